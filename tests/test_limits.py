"""Sizes beyond the documented limits are refused before any HIP call, whatever
kernel would take the call."""

import ctypes

import numpy as np
import pytest

from paper_2505_13955_amd import xct as X

ETOOBIG = -4
FAKE = ctypes.c_void_p(0x10000)


def _geom(nx, center):
    ang = np.zeros(1)
    return X.XctGeometry(1, 1, nx, 1, 1.0, 1.0, center, ang.ctypes.data_as(ctypes.POINTER(ctypes.c_double))), ang


# 2^31 work items of 64 x 64 pixels: two tiles, 2^30 slices off the half bins
# (one item per tile and slice, though slices go in pairs); four tiles and as
# many slices on them (two slices per item)
@pytest.mark.parametrize("nx, center, slices", [(65, 0.3, 1 << 30), (256, 0.0, 1 << 30), (65536, 0.3, 1 << 21)])
def test_back_projections_of_too_many_items(nx, center, slices):
    lib = X.load_library()
    g, ang = _geom(nx, center)
    gp = ctypes.byref(g)
    assert lib.xct_backproject(gp, slices, FAKE, 0, FAKE, 1.0, 0, None) == ETOOBIG
    assert lib.xct_project_adjoint(gp, slices, FAKE, FAKE, 1.0, 0, None) == ETOOBIG
    assert lib.xct_backproject_u16(gp, slices, FAKE, 0, FAKE, 1.0, 0.2, -1000.0, 3000.0, None) == ETOOBIG
    # a batch's slabs of one kernel count together
    slabs = (X.XctSlab * 2)()
    for s in slabs:
        s.geom, s.n_slices, s.sino, s.image = g, slices // 2, FAKE, FAKE
    need = lib.xct_fbp_workspace_bytes(slabs, 2, 0)
    assert need > 0
    assert lib.xct_fbp_batch(slabs, 2, 0, 0, 0, FAKE, need, None) == ETOOBIG
