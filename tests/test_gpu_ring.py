"""Backward-weights ring kernel against the oracle: chunk lengths 64 to 8,
reductions that are not a multiple of 64 (or of 32), filters and strides
beyond 3x3 same padding, at most 32 and more than 64 output channels, one and
several segments (also of an odd number of 64-index groups), columns and rows
cut by the output's edge, inputs smaller than the output grid."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, GpuLayer, note, oracle_geom, to_dev, ulp_diff
from paper_1802_00930_amd import dfp

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, c, h, w, k, r, s, stride, pad
    (2, 16, 14, 14, 32, 3, 3, 1, 1),    # 392 indices, 32 rows
    (1, 5, 5, 5, 3, 3, 3, 1, 1),        # 25 indices: one partial group
    (3, 24, 9, 11, 72, 3, 3, 1, 1),     # two row tiles, 297 indices
    (2, 3, 30, 30, 40, 7, 7, 2, 3),     # few channels, four phases (columns read one by one)
    (1, 3, 32, 32, 64, 7, 7, 2, 3),     # the same with stride-2 rows read eight columns at a time
    (2, 8, 13, 15, 16, 3, 3, 2, 1),     # stride 2, odd sizes: a phase smaller than the grid
    (1, 70, 8, 16, 33, 1, 3, 1, 1),     # 1x3 filter padded in both directions: output taller than the input
    (2, 9, 10, 10, 20, 5, 5, 1, 2),
    (2, 66, 12, 12, 64, 1, 1, 1, 0),    # 1x1 (at chunk lengths below 32)
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("L,G", [(64, 0), (64, 1), (64, 3), (32, 0), (32, 2), (16, 0), (16, 12), (8, 0), (8, 8), (8, 5)])
def test_ring(shape, L, G):
    n, c, h, w, k, r, s, st, pd = shape
    gl = GpuLayer(n, c, h, w, k, r, s, st, pd, L=L, G=G)
    rng = np.random.default_rng([n, c, h, k, r, L, G])
    x = rng.integers(-16384, 16385, gl.shape_x).astype(np.int16)
    dy = rng.integers(-16384, 16385, gl.shape_y).astype(np.int16)
    sc = torch.tensor([0, -12, 0, 0], dtype=torch.int32, device=DEV)
    note("ring shape=%s L=%d G=%d" % (shape, L, G))
    out, _, _ = gl.conv(dfp.BWD_WT, to_dev(x), sc, to_dev(dy), sc)
    ref, _, _ = oracle.conv(oracle_geom(gl), dfp.BWD_WT, x, dy, -24, L, G if G else oracle.default_seg_chunks(L))
    torch.cuda.synchronize()
    assert ulp_diff(out.cpu().numpy(), ref) == 0
