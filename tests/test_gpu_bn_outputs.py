"""Batch norm without the optional FP32 outputs: the backward call without dy
rounds with the ReLU mask that the statistics pass left in dyq (residual, hw a
multiple of four) or with the recomputed pre-activation, the forward call
without z rounds the recomputed output.  Integers and scales against the
oracle, over group counts that fill whole waves and that do not, up to tensors
of several rounds of the rounding pass's grid (8192 workgroups of 256 groups
of four elements) whose last round is partly filled."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, note, to_dev
from paper_1802_00930_amd import dfp
from test_gpu_train import bn_inputs, scale_with_exp

pytestmark = pytest.mark.gpu

# the last three: 2283336, 2131078 (the last one short) and 2098176 groups against rounds of 2097152
SHAPES = [(1, 1, 1), (2, 3, 4), (2, 6, 35), (3, 5, 49), (4, 8, 64), (5, 7, 12), (33, 72, 3844), (17, 41, 12230),
          (16, 64, 8192 + 4)]


def _case(shape, seed, with_res):
    y, ey, gamma, beta, res = bn_inputs(seed, *shape, with_res=with_res)
    dz = np.random.default_rng(seed + 1).integers(-16384, 16385, shape).astype(np.int16)
    four = lambda a: None if a is None else a.reshape(shape + (1,))
    return y, ey, gamma, beta, res, dz, four


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("with_res", [True, False])
def test_bn_integers_alone(shape, with_res):
    N, C, HW = shape
    rounding, seed = 1 if HW < 1000 else 0, 11 + N + C + HW
    y, ey, gamma, beta, res, dz, four = _case(shape, seed, with_res)
    fw = oracle.bn_relu_fwd(four(y), ey, gamma, beta, four(res), rounding=rounding, seed=seed)
    bw = oracle.bn_relu_bwd(four(dz), -24, four(y), ey, gamma, beta, fw["mean"], fw["inv_std"], four(res),
                            rounding=rounding, seed=seed)
    d = dfp.make_bn_desc(N, C, HW, rounding=rounding, seed=seed)
    ws = dfp.alloc_bn_workspace(d, DEV)
    yt, rt, g, b = to_dev(y), None if res is None else to_dev(res), to_dev(gamma), to_dev(beta)
    mean, inv, dg, db = (torch.empty(C, dtype=torch.float32, device=DEV) for _ in range(4))
    q, s = torch.empty_like(yt), dfp.new_scale(DEV)
    note("bn fwd without z %s res=%d" % (shape, with_res))
    dfp.dfp_bn_relu_fwd(d, yt, scale_with_exp(ey), g, b, q, s, mean, inv, res=rt, workspace=ws)
    sc = dfp.read_scale(s)
    assert (sc["exp"], sc["flags"]) == (fw["ez"], fw["flags"])
    assert np.count_nonzero(q.cpu().numpy().reshape(-1) != fw["zq"].reshape(-1)) == 0
    q.fill_(-1)
    note("bn bwd without dy %s res=%d" % (shape, with_res))
    dfp.dfp_bn_relu_bwd(d, to_dev(dz), scale_with_exp(-24), yt, scale_with_exp(ey), g, b, mean, inv, q, s, dg, db,
                        res=rt, workspace=ws)
    sc = dfp.read_scale(s)
    assert (sc["exp"], sc["flags"]) == (bw["edy"], bw["flags"])
    assert np.count_nonzero(q.cpu().numpy().reshape(-1) != bw["dyq"].reshape(-1)) == 0
    assert np.array_equal(dg.cpu().numpy().view(np.uint32), bw["dgamma"].view(np.uint32))
    assert np.array_equal(db.cpu().numpy().view(np.uint32), bw["dbeta"].view(np.uint32))
