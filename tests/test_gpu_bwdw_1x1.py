"""1x1 backward-weights kernel that reads the INT16 tensors, against the oracle:
pieces of 8 and of 4 indices, images smaller than a band of 64 (several per
band) and larger, bands that end past the reduction, channel counts cut by the
tiles' edges, chunks of one step and of several, segments of an odd number of
32-index blocks, unit and larger strides."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, GpuLayer, note, oracle_geom, to_dev, ulp_diff
from paper_1802_00930_amd import dfp

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, c, h, w, k, stride
    (1, 1, 2, 2, 1, 1),        # 4 indices
    (40, 20, 2, 2, 70, 1),     # 16 images a band
    (7, 65, 4, 5, 64, 1),      # 20 pixels: a band spans four images
    (3, 64, 8, 8, 128, 1),     # an image is one band
    (5, 33, 6, 6, 17, 1),      # 36 pixels
    (2, 130, 14, 14, 63, 1),
    (2, 64, 16, 18, 96, 1),    # pieces of 8
    (2, 24, 16, 16, 40, 2),
    (5, 64, 6, 6, 64, 1),      # whole tiles, the last band cut
    (3, 64, 8, 9, 128, 1),     # whole tiles, pieces of 8
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("L,G", [(64, 0), (64, 1), (64, 2), (32, 0), (32, 1), (32, 3), (96, 0), (96, 1), (128, 0),
                                 (128, 1)])
def test_bwdw_1x1(shape, L, G):
    n, c, h, w, k, st = shape
    gl = GpuLayer(n, c, h, w, k, 1, 1, st, 0, L=L, G=G)
    rng = np.random.default_rng([n, c, h, k, L, G])
    x = rng.integers(-16384, 16385, gl.shape_x).astype(np.int16)
    dy = rng.integers(-16384, 16385, gl.shape_y).astype(np.int16)
    sc = torch.tensor([0, -12, 0, 0], dtype=torch.int32, device=DEV)
    note("bwdw 1x1 shape=%s L=%d G=%d" % (shape, L, G))
    out, _, _ = gl.conv(dfp.BWD_WT, to_dev(x), sc, to_dev(dy), sc)
    ref, _, _ = oracle.conv(oracle_geom(gl), dfp.BWD_WT, x, dy, -24, L, G if G else oracle.default_seg_chunks(L))
    torch.cuda.synchronize()
    assert ulp_diff(out.cpu().numpy(), ref) == 0
