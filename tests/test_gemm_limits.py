"""GEMM reductions beyond the matrix-core kernels' 32-bit positions (offsets of 2
bytes an index into a column's digits, chunk ends of up to twice the reduction)
run on the VALU kernels, which need no workspace (no GPU)."""
import os

import pytest

from paper_1802_00930_amd import build, dfp


@pytest.mark.parametrize("m,n", [(1, 1), (1, 3), (512, 1)])
@pytest.mark.parametrize("L", [64, 1 << 29, (1 << 30) - 64])
def test_longest_matrix_core_reduction(m, n, L):
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    for k in ((1 << 30) - 1, 1 << 30, (1 << 30) + 12345, (1 << 31) - 1):
        d = dfp.make_gemm_desc(m, n, k, False, True, L)
        assert (dfp.gemm_workspace_bytes(d) > 0) == (k < 1 << 30), k
        assert (dfp.gemm_blocked_workspace_bytes(d, (1 << 31) - 64 if L == 64 else L) == 0) or k < 1 << 30


def test_rows_beyond_the_grid():
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    for m in (64 * 65535, 64 * 65535 + 1, (1 << 31) - 63, (1 << 31) - 1):
        d = dfp.make_gemm_desc(m, 1, 64, False, True, 64)
        assert (dfp.gemm_workspace_bytes(d) > 0) == (m <= 64 * 65535), m
