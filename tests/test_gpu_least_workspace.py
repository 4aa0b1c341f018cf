"""Forward and backward-data with the least workspace that calls take (the
general kernels'), where dfp_workspace_bytes asks for more: same results as the
oracle, refused a byte below, and nothing written past the bytes given."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import DEV, GpuLayer, note, oracle_geom, to_dev, ulp_diff
from paper_1802_00930_amd import dfp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,h,w,k,r,s,st,pd,L,direction,least", [
    (2, 24, 20, 20, 40, 3, 3, 1, 1, 64, dfp.FWD, 90880),        # unfolded operand with the full workspace
    (2, 48, 12, 12, 48, 5, 5, 1, 2, 16, dfp.FWD, 205312),
    (3, 20, 9, 11, 24, 1, 1, 2, 0, 64, dfp.FWD, 23552),
    (2, 40, 9, 9, 24, 1, 1, 2, 0, 64, dfp.BWD_DATA, 15872),     # on the unit-stride grid
    (1, 88, 14, 14, 90, 3, 3, 1, 1, 32, dfp.BWD_DATA, 262400),
    (4, 512, 56, 56, 128, 3, 3, 2, 1, 8, dfp.BWD_DATA, 4624896)])  # output phases
def test_least_workspace(n, c, h, w, k, r, s, st, pd, L, direction, least):
    gl = GpuLayer(n, c, h, w, k, r, s, st, pd, L=L)
    assert dfp.workspace_bytes(gl.d, direction) > least
    rng = np.random.default_rng([n, c, h, k, r, L, direction])
    fwd = direction == dfp.FWD
    a = rng.integers(-16384, 16385, gl.shape_x if fwd else gl.shape_y).astype(np.int16)
    b = rng.integers(-16384, 16385, gl.shape_w).astype(np.int16)
    ta, tb, sc = to_dev(a), to_dev(b), torch.tensor([0, -12, 0, 0], dtype=torch.int32, device=DEV)
    out = torch.empty(gl.shape_y if fwd else gl.shape_x, dtype=torch.float32, device=DEV)
    call = dfp.dfp_conv_fwd if fwd else dfp.dfp_conv_bwd_data
    room = torch.full((least + 4096,), 0x5a, dtype=torch.uint8, device=DEV)
    with pytest.raises(dfp.DfpError):
        call(gl.d, ta, sc, tb, sc, out, None, room[: least - 1])
    note("least workspace %s" % ((n, c, h, w, k, r, s, st, pd, L, direction),))
    call(gl.d, ta, sc, tb, sc, out, None, room[:least])
    ref, _, _ = oracle.conv(oracle_geom(gl), direction, a, b, -24, L)
    assert ulp_diff(out.cpu().numpy(), ref) == 0
    assert bool((room[least:] == 0x5a).all())
