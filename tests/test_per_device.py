"""Host state kept per device, on stand-ins for the HIP calls (tests/helpers/
hip_stub.c, no GPU): the ring kernel's LDS allowance is asked for once on every
device that runs it, and a device that refuses it fails the call before the
kernel is launched."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1802_00930_amd", "libdfp.so")

CHILD = """
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
dev, fails = (ctypes.c_int.in_dll(stub, n) for n in ("stub_device", "stub_attribute_fails"))
attrs, launches = ((ctypes.c_int * 64).in_dll(stub, n) for n in ("stub_attributes", "stub_launches"))
# n, c, h, w, k, r, s, strides, pads, chunk_len 16, seg_chunks, bits, rounding, path, seed (two words)
d = (ctypes.c_int32 * 18)(2, 16, 14, 14, 32, 3, 3, 1, 1, 1, 1, 16, 0, 15, 0, 0, 0, 0)
P, Z = ctypes.c_void_p, ctypes.c_size_t
lib.dfp_workspace_bytes.restype = Z
lib.dfp_workspace_bytes.argtypes = [P, ctypes.c_int32]
need = lib.dfp_workspace_bytes(d, 2)
f = lib.dfp_conv_bwd_weights
f.argtypes = [P, P, P, P, P, P, P, Z, P, P]
fake = 1 << 20
def call():
    return f(d, fake, fake, fake, fake, fake, fake, need, None, None)
for device in (0, 0, 1, 1, 0):
    dev.value = device
    assert call() == 0
assert list(attrs)[:3] == [1, 1, 0], list(attrs)[:3]
whole = launches[1] // 2  # per call
dev.value, fails.value = 2, 1
assert call() == 6, "DFP_ERR_HIP"
assert 0 < launches[2] < whole, (launches[2], whole)  # the preparation alone
fails.value = 0
assert call() == 0 and attrs[2] == 1
"""


def test_ring_lds_allowance_per_device(tmp_path):
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    stub = str(tmp_path / "hip_stub.so")
    subprocess.check_call(["gcc", "-O1", "-fPIC", "-shared", os.path.join(ROOT, "tests", "helpers", "hip_stub.c"),
                           "-o", stub])
    res = subprocess.run([sys.executable, "-c", CHILD, stub, LIB], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stderr
