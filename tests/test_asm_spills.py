"""The four-waves-per-SIMD convolution kernel at chunks below 64 has no room for
registers beyond its own: in the built assembly none of those variants spills
more than a few (a variant that also stored every chunk's partials spilled 44 to
655 and was 2 to 9 times slower than the kernels that take such calls)."""
import glob
import os
import re

import pytest

from paper_1802_00930_amd import build


def test_short_chunk_variants_keep_their_registers():
    hits = glob.glob(os.path.join(build.BUILD, "conv_mfma-hip-*.s"))
    if not hits:
        pytest.skip("library not built")
    text = open(hits[0]).read()
    found = re.findall(r"\.name: +\S*k_conv_mfma_w16ILb([01])ELb[01]ELb([01])ELi(8|16|32)E\S*.*?"
                       r"\.vgpr_spill_count: *(\d+)", text, re.S)
    assert {(phased, cl) for _, phased, cl, _ in found} == {(p, c) for p in "01" for c in ("8", "16", "32")}
    for partials, phased, cl, spills in found:
        assert int(spills) <= 8, (partials, phased, cl, spills)
