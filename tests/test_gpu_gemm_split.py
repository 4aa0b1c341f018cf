"""Split-chunk GEMM (small outputs, no partials) against the oracle: both
operands raw, either or both prepared (the four transpose settings), reductions
of one lane piece to several rounds of 16 chunks and ends inside a piece, odd
row strides, one row subtile with rows and columns cut by the edge, chunks of
32, 64 and 192, operands at 2-byte alignment; the Blocked-DFP form."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, note, to_dev, ulp_diff
from paper_1802_00930_amd import dfp

pytestmark = pytest.mark.gpu

SHAPES = [(1, 10, 65), (16, 16, 128), (17, 33, 190), (5, 300, 1025), (64, 1000, 333), (70, 500, 2050), (130, 700, 96)]


def scale(exp):
    return torch.tensor([0, exp, 0, 0], dtype=torch.int32, device=DEV)


def shifted(a):
    """The tensor at an address that is 2-byte aligned only."""
    flat = torch.zeros(a.size + 1, dtype=torch.int16, device=DEV)
    flat[1:] = to_dev(a.reshape(-1))
    return flat[1:].view(a.shape)


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("ta,tb", [(False, True), (False, False), (True, True), (True, False)])
@pytest.mark.parametrize("L", [32, 64, 192])
def test_split(m, n, k, ta, tb, L):
    rng = np.random.default_rng([m, n, k, ta, tb, L])
    a = rng.integers(-16384, 16385, (k, m) if ta else (m, k)).astype(np.int16)
    b = rng.integers(-16384, 16385, (n, k) if tb else (k, n)).astype(np.int16)
    d = dfp.make_gemm_desc(m, n, k, ta, tb, L)
    out = torch.empty(m, n, dtype=torch.float32, device=DEV)
    sd = torch.full((4,), 0x7777, dtype=torch.int32, device=DEV)
    note("gemm split %s ta=%d tb=%d L=%d" % ((m, n, k), ta, tb, L))
    put = shifted if (m + L) % 2 else to_dev
    dfp.dfp_gemm(d, put(a), scale(-11), put(b), scale(-9), out, sd, dfp.alloc_gemm_workspace(d, DEV))
    ref, _, _ = oracle.gemm(a, b, -20, L, ta, tb)
    torch.cuda.synchronize()
    assert ulp_diff(out.cpu().numpy(), ref) == 0
    assert dfp.read_scale(sd)["amax_bits"] == int((ref.view(np.uint32) & 0x7fffffff).max())


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("L,bk", [(32, 32), (64, 128), (64, 192)])
def test_split_blocked(m, n, k, L, bk):
    rng = np.random.default_rng([m, n, k, L, bk])
    nb = -(-k // bk)
    a, b = (rng.integers(-16384, 16385, (r, k)).astype(np.int16) for r in (m, n))
    ea, eb = (rng.integers(-30, 5, (nb, r)).astype(np.int8) for r in (m, n))
    d = dfp.make_gemm_desc(m, n, k, False, True, L)
    out = torch.empty(m, n, dtype=torch.float32, device=DEV)
    sd = dfp.new_scale(DEV)
    dfp.dfp_gemm_blocked(d, bk, to_dev(a), to_dev(ea), to_dev(b), to_dev(eb), out, sd,
                         dfp.alloc_gemm_blocked_workspace(d, bk, DEV))
    ref, _, _ = oracle.gemm_blocked(a, ea, b, eb, bk, L)
    torch.cuda.synchronize()
    assert ulp_diff(out.cpu().numpy(), ref) == 0
    assert dfp.read_scale(sd)["amax_bits"] == int((ref.view(np.uint32) & 0x7fffffff).max())
