"""Which route forward and backward-data take, by the workspace they ask for (no
GPU): layers measured faster with the unfolded operand or the output phases ask
for more than the general kernels', layers measured slower do not."""
import pytest

from paper_1802_00930_amd import build, dfp


@pytest.fixture(scope="module", autouse=True)
def _built():
    import os
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")


def need(n, c, h, w, k, r, st, pd, L, direction):
    return dfp.workspace_bytes(dfp.make_desc(n, c, h, w, k, r, r, st, pd, chunk_len=L), direction)


# us on an MI355X, general kernels / unfolded operand
@pytest.mark.parametrize("layer,direction,general,unfolded", [
    ((64, 32, 112, 112, 64, 3, 1, 1, 16), dfp.FWD, 282, 382),
    ((2, 80, 118, 118, 8, 7, 1, 3, 16), dfp.FWD, 194, 287),
    ((36, 48, 35, 35, 176, 7, 1, 3, 16), dfp.BWD_DATA, 502, 762),
    ((61, 144, 74, 74, 16, 3, 1, 1, 16), dfp.FWD, 468, 650),
    ((3, 16, 88, 88, 272, 3, 1, 1, 16), dfp.BWD_DATA, 126, 184),
    ((1, 16, 7, 7, 256, 3, 2, 1, 16), dfp.FWD, 14.5, 10.1),
    ((8, 16, 17, 93, 368, 1, 1, 0, 16), dfp.BWD_DATA, 67, 28),
    ((60, 16, 58, 58, 80, 1, 1, 0, 16), dfp.BWD_DATA, 61, 36),
    ((64, 88, 28, 28, 96, 3, 1, 1, 64), dfp.FWD, 272, 61)])
def test_unfolded_operand(layer, direction, general, unfolded):
    # a chunk length that the unfolded operand's kernels do not take
    plain = need(*layer[:-1], 24, direction)
    assert (need(*layer, direction) > plain) == (unfolded < general)


# us of backward-data: one dilated pass / output phases
@pytest.mark.parametrize("layer,dilated,phases", [
    ((8, 128, 28, 28, 128, 3, 2, 1, 32), 20, 57), ((32, 512, 14, 14, 64, 3, 2, 1, 32), 24, 91),
    ((8, 512, 28, 28, 64, 3, 2, 1, 16), 33, 74), ((1, 512, 14, 14, 64, 3, 2, 1, 8), 45, 55),
    ((32, 512, 56, 56, 64, 5, 2, 2, 8), 1192, 587), ((32, 512, 56, 56, 64, 5, 2, 2, 32), 409, 323)])
def test_output_phases(layer, dilated, phases):
    plain = need(*layer[:-1], 24, dfp.BWD_DATA)
    assert (need(*layer, dfp.BWD_DATA) > plain) == (phases < dilated)
