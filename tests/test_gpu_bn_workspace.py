"""Batch norm of few channels over large planes: the workspace has room for the
max pass's workgroups over the whole tensor, and a call with less (the sums and
the per-channel values alone) gives the same integers; both against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, note, to_dev
from paper_1802_00930_amd import dfp
from test_gpu_train import bn_inputs, scale_with_exp

pytestmark = pytest.mark.gpu


# (N, C, HW), bytes of the sums and the per-channel values
@pytest.mark.parametrize("shape,least", [((1, 1, 600000), 512), ((1, 16, 40000), 768), ((3, 5, 70001), 768),
                                         ((1, 2, 513), 512)])
def test_bn_workspace_room(shape, least):
    N, C, HW = shape
    y, ey, gamma, beta, res = bn_inputs(HW, N, C, HW, with_res=True)
    dz = np.random.default_rng(HW).integers(-16384, 16385, shape).astype(np.int16)
    four = lambda a: a.reshape(shape + (1,))
    fw = oracle.bn_relu_fwd(four(y), ey, gamma, beta, four(res))
    bw = oracle.bn_relu_bwd(four(dz), -24, four(y), ey, gamma, beta, fw["mean"], fw["inv_std"], four(res))
    d = dfp.make_bn_desc(N, C, HW)
    groups = min(2048, (N * C * HW + 1023) // 1024)  # of the max pass: a word each
    assert dfp.bn_workspace_bytes(d) >= (least + 4 * groups if 4 * groups > 512 else least)
    yt, rt, g, b, dzt = to_dev(y), to_dev(res), to_dev(gamma), to_dev(beta), to_dev(dz)
    mean, inv, dg, db = (torch.empty(C, dtype=torch.float32, device=DEV) for _ in range(4))
    q, s = torch.empty_like(yt), dfp.new_scale(DEV)
    for size in (dfp.bn_workspace_bytes(d), least):
        room = torch.full((size + 4096,), 0x5a, dtype=torch.uint8, device=DEV)
        note("bn workspace %s %d" % (shape, size))
        dfp.dfp_bn_relu_fwd(d, yt, scale_with_exp(ey), g, b, q, s, mean, inv, res=rt, workspace=room[:size])
        assert dfp.read_scale(s)["exp"] == fw["ez"] and np.array_equal(q.cpu().numpy().ravel(), fw["zq"].ravel())
        dfp.dfp_bn_relu_bwd(d, dzt, scale_with_exp(-24), yt, scale_with_exp(ey), g, b, mean, inv, q, s, dg, db,
                            res=rt, workspace=room[:size])
        assert dfp.read_scale(s)["exp"] == bw["edy"] and np.array_equal(q.cpu().numpy().ravel(), bw["dyq"].ravel())
        assert bool((room[size:] == 0x5a).all())
    with pytest.raises(dfp.DfpError):
        dfp.dfp_bn_relu_fwd(d, yt, scale_with_exp(ey), g, b, q, s, mean, inv, res=rt, workspace=room[: least - 1])
