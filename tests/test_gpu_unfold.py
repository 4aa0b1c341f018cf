"""Forward and backward-data of layers whose channel counts the plane layout does
not take (unfolded operand), against the oracle: channel counts off 16 and 32,
reductions past and at multiples of 64, chunks spanning filter taps, strides,
paddings, more blocks than one phase holds, few and many output rows."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, GpuLayer, note, oracle_geom, to_dev, ulp_diff
from paper_1802_00930_amd import dfp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,h,w,k,r,s,st,pd", [
    (2, 24, 9, 8, 40, 3, 3, 1, 1), (1, 88, 7, 7, 90, 3, 3, 1, 1), (2, 5, 6, 11, 7, 3, 3, 2, 1),
    (3, 72, 5, 5, 136, 1, 1, 1, 0), (2, 40, 9, 9, 24, 1, 1, 2, 0), (1, 17, 8, 6, 33, 5, 3, 1, 2),
    (1, 200, 6, 6, 130, 3, 3, 1, 1), (2, 16, 7, 7, 48, 3, 3, 1, 1), (1, 1, 3, 3, 1, 2, 2, 1, 0),
    (1, 1000, 4, 4, 520, 1, 1, 1, 0)])
@pytest.mark.parametrize("L", [64, 32, 16, 8])
@pytest.mark.parametrize("direction", [dfp.FWD, dfp.BWD_DATA])
def test_unfold(n, c, h, w, k, r, s, st, pd, L, direction):
    gl = GpuLayer(n, c, h, w, k, r, s, st, pd, L=L)
    rng = np.random.default_rng([n, c, h, k, r, L, direction])
    src = rng.integers(-16384, 16385, gl.shape_x if direction == dfp.FWD else gl.shape_y).astype(np.int16)
    wt = rng.integers(-16384, 16385, gl.shape_w).astype(np.int16)
    sc = torch.tensor([0, -12, 0, 0], dtype=torch.int32, device=DEV)
    note("unfold %s L=%d dir=%d" % ((n, c, h, w, k, r, s, st, pd), L, direction))
    out, so, _ = gl.conv(direction, to_dev(src), sc, to_dev(wt), sc)
    ref, _, _ = oracle.conv(oracle_geom(gl), direction, src, wt, -24, L)
    torch.cuda.synchronize()
    assert ulp_diff(out.cpu().numpy(), ref) == 0
    assert dfp.read_scale(so)["amax_bits"] == int((np.abs(ref).astype(np.float32).view(np.uint32)).max())


def test_unfold_large_filter():
    """More filter items than one row of workgroups per grid row can take."""
    gl = GpuLayer(1, 8191, 1, 1, 8256, 1, 1, 1, 0, L=64)
    rng = np.random.default_rng(3)
    x = rng.integers(-16384, 16385, gl.shape_x).astype(np.int16)
    wt = rng.integers(-16384, 16385, gl.shape_w, dtype=np.int16)
    sc = torch.tensor([0, -12, 0, 0], dtype=torch.int32, device=DEV)
    note("unfold large filter")
    out, _, _ = gl.conv(dfp.FWD, to_dev(x), sc, to_dev(wt), sc)
    ref, _, _ = oracle.conv(oracle_geom(gl), dfp.FWD, x, wt, -24, 64)
    torch.cuda.synchronize()
    assert ulp_diff(out.cpu().numpy(), ref) == 0
