"""Backward-weights layers with rows too wide for the general matrix-core
kernel's band: with a workspace (1x1 kernels, ring kernel), without one and with
partials (VALU kernel), and through the entry point without a workspace argument,
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, GpuLayer, note, oracle_geom, to_dev, ulp_diff
from paper_1802_00930_amd import dfp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,h,w,k,r,st,pd", [(1, 130, 9, 140, 24, 1, 1, 0), (2, 128, 9, 99, 17, 1, 1, 0),
                                               (1, 129, 17, 198, 8, 1, 2, 0), (3, 200, 9, 104, 70, 1, 1, 0)])
@pytest.mark.parametrize("L", [64, 32, 16, 8, 24])
def test_bwdw_wide(n, c, h, w, k, r, st, pd, L):
    gl = GpuLayer(n, c, h, w, k, r, r, st, pd, L=L)
    d = gl.d
    rng = np.random.default_rng([n, c, h, k, r, L])
    x = rng.integers(-16384, 16385, gl.shape_x).astype(np.int16)
    dy = rng.integers(-16384, 16385, gl.shape_y).astype(np.int16)
    sc = torch.tensor([0, -12, 0, 0], dtype=torch.int32, device=DEV)
    note("bwdw wide %s L=%d" % ((n, c, h, w, k, r, st, pd), L))
    J = int(dfp.num_chunks(d, dfp.BWD_WT))
    ref, rparts, _ = oracle.conv(oracle_geom(gl), dfp.BWD_WT, x, dy, -24, L, oracle.default_seg_chunks(L),
                                 want_partials=True)
    xt, dyt = to_dev(x), to_dev(dy)
    calls = {
        "workspace": lambda o: dfp.dfp_conv_bwd_weights(d, xt, sc, dyt, sc, o, dfp.alloc_workspace(d, dfp.BWD_WT)),
        "noalloc": lambda o: dfp.dfp_conv_bwd_weights_noalloc(d, xt, sc, dyt, sc, o),
    }
    if L != 24:
        assert dfp.workspace_bytes(d, dfp.BWD_WT) > 0
        calls["no workspace"] = lambda o: dfp.dfp_conv_bwd_weights(d, xt, sc, dyt, sc, o, None)
    for name, call in calls.items():
        out = torch.full(gl.shape_w, 7.0, device=DEV)
        call(out)
        torch.cuda.synchronize()
        assert ulp_diff(out.cpu().numpy(), ref) == 0, name
    parts = torch.empty((J,) + tuple(gl.shape_w), dtype=torch.int32, device=DEV)
    dfp.dfp_conv_bwd_weights(d, xt, sc, dyt, sc, out, dfp.alloc_workspace(d, dfp.BWD_WT), partials=parts)
    torch.cuda.synchronize()
    assert np.array_equal(parts.cpu().numpy().reshape(-1), np.asarray(rparts).reshape(-1))
    assert ulp_diff(out.cpu().numpy(), ref) == 0
