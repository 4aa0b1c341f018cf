"""P = 16 convolutions on the matrix cores: tensors whose integers all fit the
byte digits (at most 32639), tensors with larger ones in the first operand, in
the second or in the very last element (the gated VALU kernels then compute
the output), without a workspace (VALU alone) and from a 2-byte aligned
tensor.  FP32 outputs 0 ulp from the oracle, the output scale exact."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, GpuLayer, note, oracle_geom, to_dev, ulp_diff
from paper_1802_00930_amd import dfp

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, c, h, w, k, r, s, stride, pad
    (2, 16, 14, 14, 32, 3, 3, 1, 1),
    (1, 3, 23, 23, 8, 7, 7, 2, 3),
    (2, 64, 9, 11, 40, 3, 3, 1, 1),
    (1, 96, 8, 8, 130, 1, 1, 1, 0),
    (2, 64, 10, 10, 64, 1, 1, 2, 0),
    (1, 32, 9, 9, 64, 3, 3, 2, 1),
]


def scale(exp):
    return torch.tensor([0, exp, 0, 0], dtype=torch.int32, device=DEV)


def operand(rng, shape, beyond):
    a = rng.integers(-32767, 32640, shape).astype(np.int16)
    a.reshape(-1)[:2] = (32639, -32767)
    if beyond == "some":
        a.reshape(-1)[rng.integers(0, a.size, 5)] = rng.integers(32640, 32768, 5)
    elif beyond == "last":
        a.reshape(-1)[-1] = 32640
    return a


def roles(gl, direction):
    return {dfp.FWD: (gl.shape_x, gl.shape_w), dfp.BWD_DATA: (gl.shape_y, gl.shape_w),
            dfp.BWD_WT: (gl.shape_x, gl.shape_y)}[direction]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("beyond", [(None, None), ("some", None), (None, "last"), ("last", "some")])
@pytest.mark.parametrize("L", [16, 20, 64])
def test_p16_conv(shape, beyond, L):
    n, c, h, w, k, r, s, st, pd = shape
    gl = GpuLayer(n, c, h, w, k, r, s, st, pd, L=L, bits=16)
    rng = np.random.default_rng([n, c, h, w, k, r, L, beyond[0] is not None, beyond[1] is not None])
    for direction in (dfp.FWD, dfp.BWD_DATA, dfp.BWD_WT):
        sa, sb = roles(gl, direction)
        a, b = operand(rng, sa, beyond[0]), operand(rng, sb, beyond[1])
        note("p16 shape=%s L=%d dir=%d beyond=%s" % (shape, L, direction, beyond))
        assert dfp.workspace_bytes(gl.d, direction) > 0
        out, so, _ = gl.conv(direction, to_dev(a), scale(-14), to_dev(b), scale(-15))
        ref, _, _ = oracle.conv(oracle_geom(gl), direction, a, b, -29, L, oracle.default_seg_chunks(L))
        torch.cuda.synchronize()
        assert ulp_diff(out.cpu().numpy(), ref) == 0
        if so is not None:
            info = dfp.read_scale(so)
            assert info["amax_bits"] == int((ref.view(np.uint32) & 0x7fffffff).max()) and info["flags"] == 0


@pytest.mark.parametrize("beyond", [None, "some"])
def test_p16_conv_i32(beyond):
    n, c, h, w, k, r, s, st, pd = SHAPES[2]
    rng = np.random.default_rng(5)
    for direction, T in ((dfp.FWD, c * r * s), (dfp.BWD_DATA, k * r * s)):
        gl = GpuLayer(n, c, h, w, k, r, s, st, pd, L=T, bits=16)
        sa, sb = roles(gl, direction)
        a, b = operand(rng, sa, beyond), operand(rng, sb, None)
        out = torch.zeros(gl.shape_y if direction == dfp.FWD else gl.shape_x, dtype=torch.int32, device=DEV)
        so = torch.full((4,), 0x1234, dtype=torch.int32, device=DEV)
        call = dfp.dfp_conv_fwd_i32 if direction == dfp.FWD else dfp.dfp_conv_bwd_data_i32
        call(gl.d, to_dev(a), scale(-3), to_dev(b), scale(-4), out, so, dfp.alloc_workspace(gl.d, direction, DEV))
        _, parts, _ = oracle.conv(oracle_geom(gl), direction, a, b, -7, T, 1, want_partials=True)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().reshape(-1), parts[0])
        info = dfp.read_scale(so)
        assert info == {"amax_bits": int(np.abs(parts[0].astype(np.int64)).max()), "exp": -7, "flags": 0}


@pytest.mark.parametrize("beyond", [None, "some"])
def test_p16_without_workspace_and_misaligned(beyond):
    gl = GpuLayer(*SHAPES[0], L=16, bits=16)
    rng = np.random.default_rng(6)
    a, b = operand(rng, gl.shape_x, beyond), operand(rng, gl.shape_w, None)
    ref, _, _ = oracle.conv(oracle_geom(gl), oracle.FWD, a, b, 0, 16)
    flat = torch.zeros(a.size + 1, dtype=torch.int16, device=DEV)
    flat[1:] = to_dev(a.reshape(-1))
    for x, ws in ((to_dev(a), None), (flat[1:], dfp.alloc_workspace(gl.d, dfp.FWD, DEV))):
        y = torch.empty(gl.shape_y, dtype=torch.float32, device=DEV)
        dfp.dfp_conv_fwd(gl.d, x, scale(0), to_dev(b), scale(0), y, None, ws)
        torch.cuda.synchronize()
        assert ulp_diff(y.cpu().numpy(), ref) == 0
