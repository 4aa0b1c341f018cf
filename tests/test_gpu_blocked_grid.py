"""Blocked quantiser past the grid of 4096 waves (grid-stride loop, several
groups per lane) and the tensor's zero flag when only its last row, or none, is
non-zero: integers, exponents, max and flags equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import note
from paper_1802_00930_amd import dfp
from test_gpu_blocked import quantize_blocked_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,B", [((8300, 128), 16), ((2100, 512), 64), ((1100, 2052), 516)])  # 4150 to 4400 waves
@pytest.mark.parametrize("fill", ["dense", "last row"])
def test_quantize_blocked_grid_stride(shape, B, fill):
    note("quantize_blocked grid %s B=%d %s" % (shape, B, fill))
    f = np.random.default_rng([shape[0], B]).standard_normal(shape).astype(np.float32)
    if fill == "last row":
        f[:-1] = 0.0
    q, e, sc = quantize_blocked_gpu(f, B, 15, "stochastic", 77, dfp.ROLE_X)
    rq, re, rfl = oracle.quantize_blocked(f, B, 15, oracle.ROUND_STOCHASTIC, 77, dfp.ROLE_X)
    torch.cuda.synchronize()
    assert np.array_equal(q.cpu().numpy(), rq) and np.array_equal(e.cpu().numpy(), re)
    s = dfp.read_scale(sc)
    assert s["flags"] == rfl and s["amax_bits"] == int((f.view(np.uint32) & 0x7fffffff).max())
