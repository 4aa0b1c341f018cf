"""Unfolded operand where the plain layout of the same input is 2 GiB or more
(large strides over many pixels): images at both ends and in the middle against
the oracle, which takes an image at a time."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, GpuLayer, note, oracle_geom, ulp_diff
from paper_1802_00930_amd import dfp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,h,w,k,r,st,L", [
    (300, 3, 500, 480, 20, 4, 16, 64),  # plain 2.30e9 bytes in 16-channel groups, unfolded 0.04e9
    (300, 17, 400, 480, 33, 2, 8, 16),  # plain 3.7e9, unfolded 0.23e9
])
def test_unfold_beyond_plain_2gib(n, c, h, w, k, r, st, L):
    gl = GpuLayer(n, c, h, w, k, r, r, st, 0, L=L)
    one = GpuLayer(1, c, h, w, k, r, r, st, 0, L=L)
    assert dfp.workspace_bytes(gl.d, dfp.FWD) >= 1 << 31
    gen = torch.Generator(device=DEV).manual_seed(c)
    x = torch.randint(-16384, 16385, gl.shape_x, generator=gen, device=DEV, dtype=torch.int16)
    wt = torch.randint(-16384, 16385, gl.shape_w, generator=gen, device=DEV, dtype=torch.int16)
    sc = torch.tensor([0, -12, 0, 0], dtype=torch.int32, device=DEV)
    note("unfold, plain layout of 2 GiB: %s" % ((n, c, h, w, k, r, st, L),))
    out, _, _ = gl.conv(dfp.FWD, x, sc, wt, sc)
    for i in (0, 1, n // 2, n - 1):
        ref, _, _ = oracle.conv(oracle_geom(one), dfp.FWD, x[i: i + 1].cpu().numpy(), wt.cpu().numpy(), -24, L)
        assert ulp_diff(out[i].cpu().numpy(), ref) == 0, i
