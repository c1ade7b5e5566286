"""Cell lists, their counts and the kernels' cell and face numbers have 32 bits: adg_create takes fewer than
2^31 cells (host side, no GPU)."""
import ctypes

import pytest

from paper_1406_7416_amd import adg
from paper_1406_7416_amd import workloads as W


@pytest.mark.parametrize("ncell,accepted", [((1 << 16, 1 << 15), False), ((1 << 30, 2), False),
                                            ((1 << 16, (1 << 15) - 1), True), (((1 << 30) - 1, 2), True)])
def test_fewer_than_2_31_cells(ncell, accepted):
    L = adg.load()
    wl = W.explosion_2d(8, 1)
    wl.ncell = ncell
    grid, prm, h = adg._grid(wl), adg._Params(), ctypes.c_void_p()
    prm.limiter = 1
    rc = L.adg_create(ctypes.byref(grid), 1, 1.4, ctypes.byref(prm), ctypes.byref(h))
    assert rc == (0 if accepted else -1)
    if accepted:
        assert L.adg_workspace_bytes(h) > 0
        L.adg_destroy(h)
