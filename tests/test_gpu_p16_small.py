"""P = 16 layers on both sides of the line below which path AUTO keeps the VALU
kernels: AUTO and MFMA (always the matrix cores behind the scan), integers within
the byte digits and beyond, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GpuLayer, note, oracle_geom, to_dev, ulp_diff
from paper_1802_00930_amd import dfp
from test_gpu_p16 import operand, roles, scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 3, 3, 1, 1, 1, 1, 0), (1, 8, 7, 7, 8, 3, 3, 1, 1), (1, 16, 7, 7, 16, 1, 1, 1, 0),
                                   (2, 48, 9, 9, 40, 3, 3, 2, 1), (4, 40, 15, 15, 40, 3, 3, 1, 1)])
@pytest.mark.parametrize("path", [dfp.PATH_AUTO, dfp.PATH_MFMA])
@pytest.mark.parametrize("L", [16, 20])
@pytest.mark.parametrize("beyond", [None, "last"])
def test_p16_small(shape, path, L, beyond):
    n, c, h, w, k, r, s, st, pd = shape
    gl = GpuLayer(n, c, h, w, k, r, s, st, pd, L=L, bits=16, path=path)
    rng = np.random.default_rng([n, c, h, k, r, L, path])
    for direction in (dfp.FWD, dfp.BWD_DATA, dfp.BWD_WT):
        sa, sb = roles(gl, direction)
        a, b = operand(rng, sa, beyond) if np.prod(sa) > 2 else rng.integers(-9, 9, sa).astype(np.int16), \
            rng.integers(-32767, 32640, sb).astype(np.int16)
        note("p16 small %s path=%d L=%d dir=%d beyond=%s" % (shape, path, L, direction, beyond))
        out, so, _ = gl.conv(direction, to_dev(a), scale(-14), to_dev(b), scale(-15))
        ref, _, _ = oracle.conv(oracle_geom(gl), direction, a, b, -29, L, oracle.default_seg_chunks(L))
        torch.cuda.synchronize()
        assert ulp_diff(out.cpu().numpy(), ref) == 0
        if so is not None:
            assert dfp.read_scale(so)["amax_bits"] == int((ref.view(np.uint32) & 0x7fffffff).max())
