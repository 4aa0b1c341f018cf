"""Blocked quantiser over numbers of waves around the steps of its workgroup size
(one wave per block of 256 elements, 1 to 16 waves a workgroup, at most 256
workgroups), last rounds around the three quarters of 4096 waves below which they
are dealt over the workgroups, and block lengths around the two-groups-per-lane
line: integers, exponents, max and flags equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import note
from paper_1802_00930_amd import dfp
from test_gpu_blocked import quantize_blocked_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,B", [((1, 256), 256), ((255, 256), 256), ((257, 256), 256), ((513, 256), 256),
                                     ((3841, 256), 256), ((4097, 256), 256), ((7168, 256), 256), ((7169, 256), 256),
                                     ((8191, 256), 256), ((4300, 63), 63), ((7200, 63), 63), ((3, 1536), 512), ((5, 2064), 516),
                                     ((2, 70000), 70000), ((3, 4999), 4999), ((7, 33), 5)])
@pytest.mark.parametrize("rounding", ["nearest", "stochastic"])
def test_quantize_blocked_waves(shape, B, rounding):
    note("quantize_blocked waves %s B=%d %s" % (shape, B, rounding))
    f = np.random.default_rng([shape[0], shape[1], B]).standard_normal(shape).astype(np.float32)
    f[shape[0] // 2] *= 1e-3
    f[-1, : B] = 0.0
    q, e, sc = quantize_blocked_gpu(f, B, 15, rounding, 77, dfp.ROLE_X)
    rq, re, rfl = oracle.quantize_blocked(f, B, 15, oracle.ROUND_STOCHASTIC if rounding == "stochastic" else 0, 77,
                                          dfp.ROLE_X)
    torch.cuda.synchronize()
    assert np.array_equal(q.cpu().numpy(), rq) and np.array_equal(e.cpu().numpy(), re)
    s = dfp.read_scale(sc)
    assert s["flags"] == rfl and s["amax_bits"] == int((f.view(np.uint32) & 0x7fffffff).max())
