"""Chunks below 64 on the routes that the plan takes by its estimates: output
phases of strided backward-data and the unfolded operand over channels in whole
groups of 16.  The workspace says that the layer takes the route; outputs at
sampled positions (every phase among them) and the output scale against the
oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, GpuLayer, note, oracle_geom, to_dev, ulp_diff
from paper_1802_00930_amd import dfp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,h,w,k,r,st,pd,L,direction", [
    (4, 512, 56, 56, 128, 3, 2, 1, 8, dfp.BWD_DATA), (2, 512, 56, 55, 128, 5, 2, 2, 16, dfp.BWD_DATA),
    (2, 512, 55, 56, 128, 5, 2, 2, 32, dfp.BWD_DATA),
    (1, 16, 10, 10, 48, 5, 1, 2, 16, dfp.FWD), (1, 16, 12, 9, 48, 5, 1, 2, 8, dfp.FWD),
    (1, 48, 10, 11, 16, 5, 1, 2, 16, dfp.BWD_DATA), (2, 80, 9, 9, 33, 1, 1, 0, 8, dfp.FWD)])
def test_short_chunk_route(n, c, h, w, k, r, st, pd, L, direction):
    gl = GpuLayer(n, c, h, w, k, r, r, st, pd, L=L)
    general = dfp.make_desc(n, c, h, w, k, r, r, st, pd, chunk_len=24)
    assert dfp.workspace_bytes(gl.d, direction) > dfp.workspace_bytes(general, direction)
    rng = np.random.default_rng([n, c, h, k, r, L, direction])
    src = rng.integers(-16384, 16385, gl.shape_x if direction == dfp.FWD else gl.shape_y).astype(np.int16)
    wt = rng.integers(-16384, 16385, gl.shape_w).astype(np.int16)
    sc = torch.tensor([0, -12, 0, 0], dtype=torch.int32, device=DEV)
    note("short route %s L=%d dir=%d" % ((n, c, h, w, k, r, st, pd), L, direction))
    out, so, _ = gl.conv(direction, to_dev(src), sc, to_dev(wt), sc)
    flat = out.cpu().numpy().reshape(-1)
    idx = np.unique(np.concatenate([np.arange(min(3 * w, flat.size)), np.arange(max(0, flat.size - 3 * w), flat.size),
                                    rng.integers(0, flat.size, 4000)]))
    ref, _, _ = oracle.conv_at(oracle_geom(gl), direction, src, wt, -24, L, idx)
    assert ulp_diff(flat[idx], ref) == 0
    assert dfp.read_scale(so)["amax_bits"] == int((flat.view(np.uint32) & 0x7fffffff).max())
