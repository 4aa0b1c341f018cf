"""Split-chunk GEMM with two and four row subtiles per workgroup (outputs of more
than 320 and 600 tiles of 16 x 16), and with operands whose rows are not 4-byte
aligned: prepared where several workgroups read them, as INT16 where one does;
also the Blocked-DFP form.  Against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, note, to_dev, ulp_diff
from paper_1802_00930_amd import dfp
from test_gpu_gemm_split import scale, shifted

pytestmark = pytest.mark.gpu

SHAPES = [(130, 700, 1000), (130, 700, 1001), (200, 1000, 1030), (201, 1003, 1031), (3, 800, 1033), (700, 9, 1035)]


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("ta,tb", [(False, True), (False, False), (True, True), (True, False)])
@pytest.mark.parametrize("L", [32, 64])
@pytest.mark.parametrize("put", [to_dev, shifted])
def test_split_wide(m, n, k, ta, tb, L, put):
    rng = np.random.default_rng([m, n, k, ta, tb, L])
    a = rng.integers(-16384, 16385, (k, m) if ta else (m, k)).astype(np.int16)
    b = rng.integers(-16384, 16385, (n, k) if tb else (k, n)).astype(np.int16)
    d = dfp.make_gemm_desc(m, n, k, ta, tb, L)
    out, sd = torch.empty(m, n, dtype=torch.float32, device=DEV), dfp.new_scale(DEV)
    note("gemm split wide %s ta=%d tb=%d L=%d" % ((m, n, k), ta, tb, L))
    dfp.dfp_gemm(d, put(a), scale(-11), put(b), scale(-9), out, sd, dfp.alloc_gemm_workspace(d, DEV))
    ref, _, _ = oracle.gemm(a, b, -20, L, ta, tb)
    assert ulp_diff(out.cpu().numpy(), ref) == 0
    assert dfp.read_scale(sd)["amax_bits"] == int((ref.view(np.uint32) & 0x7fffffff).max())


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("L,bk", [(32, 64), (64, 128)])
@pytest.mark.parametrize("put", [to_dev, shifted])
def test_split_wide_blocked(m, n, k, L, bk, put):
    rng = np.random.default_rng([m, n, k, L, bk])
    nb = -(-k // bk)
    a, b = (rng.integers(-16384, 16385, (r, k)).astype(np.int16) for r in (m, n))
    ea, eb = (rng.integers(-30, 5, (nb, r)).astype(np.int8) for r in (m, n))
    d = dfp.make_gemm_desc(m, n, k, False, True, L)
    out, sd = torch.empty(m, n, dtype=torch.float32, device=DEV), dfp.new_scale(DEV)
    note("gemm split wide blocked %s L=%d" % ((m, n, k), L))
    dfp.dfp_gemm_blocked(d, bk, put(a), to_dev(ea), put(b), to_dev(eb), out, sd,
                         dfp.alloc_gemm_blocked_workspace(d, bk, DEV))
    ref, _, _ = oracle.gemm_blocked(a, ea, b, eb, bk, L)
    assert ulp_diff(out.cpu().numpy(), ref) == 0
    assert dfp.read_scale(sd)["amax_bits"] == int((ref.view(np.uint32) & 0x7fffffff).max())
