"""The 1x1 backward-weights kernel reads the caller's tensors with buffer loads
and sends rows and indices past their end to an offset that the range check
refuses.  That check covers the vector offset; in the built assembly of the
variants for row counts that are not whole tiles the loads must therefore carry
no scalar offset."""
import glob
import os
import re

import pytest

from paper_1802_00930_amd import build


def test_1x1_loads_have_no_scalar_offset():
    hits = glob.glob(os.path.join(build.BUILD, "conv_bwdw_mfma-hip-*.s"))
    if not hits:
        pytest.skip("library not built")
    text = open(hits[0]).read()
    kernels = re.findall(r"^(_ZN\S*k_bwdw_1x1sILi[48]ELi\d+ELb[01]ELb1\S*):(.*?)\.Lfunc_end", text, re.S | re.M)
    assert len(kernels) == 8  # pieces of 8 and 4, 64 and 32 indices a step, one or more steps a chunk
    for name, body in kernels:
        loads = re.findall(r"buffer_load_\w+ +[^,]+, *v\d+, *s\[\d+:\d+\], *(\S+) offen", body)
        assert loads and set(loads) == {"0"}, (name, loads)
