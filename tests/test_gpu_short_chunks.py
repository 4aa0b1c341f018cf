"""Forward and backward-data at chunk lengths 8, 16 and 32 on the
four-waves-per-SIMD kernel: one filter phase (2 to 36 blocks), several phases,
row tiles cut by the output channels, tiles cut by the pixels, stride 2, and with
partials (on the masked and shared-ring kernels), against the oracle."""
import pytest

from paper_1802_00930_amd import dfp
from test_gpu_conv import run_all

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, c, h, w, k, r, s, stride, pad
    (1, 64, 5, 7, 32, 1, 1, 1, 0),     # 2 blocks, 35 pixels
    (2, 32, 9, 11, 64, 4, 4, 1, 2),    # 16 blocks, 4x4 taps
    (1, 128, 6, 6, 96, 3, 3, 1, 1),    # 36 blocks
    (1, 256, 7, 7, 72, 3, 3, 1, 1),    # two phases, a cut row tile
    (2, 64, 9, 9, 128, 3, 3, 2, 1),    # stride 2: backward over the dilated gradient
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("L", [8, 16, 32])
@pytest.mark.parametrize("partials", [False, True])
@pytest.mark.parametrize("path", [dfp.PATH_AUTO, dfp.PATH_MFMA])
def test_short_chunks(shape, L, partials, path):
    run_all(shape, L, path=path, partials=partials)
