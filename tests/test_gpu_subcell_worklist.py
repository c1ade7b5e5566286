"""The subcell recompute where workgroups take several troubled cells one after the other in the mixed form,
and at 3D N = 9 (19^3 subcells, 9025 positions), against the FP64 oracle, every step compared.

Tolerances of the other parity tests: FP64 1e-12 of each variable's scale on the first step, 1e-10 after,
identical troubled maps; mixed form 2e-6.
"""
import numpy as np
import pytest

from paper_1406_7416_amd import workloads as W
from test_gpu_mixed import paired_mixed, run_mixed
from test_gpu_parity import paired, run_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 3])
def test_several_cells_per_workgroup_mixed(N):
    """37 x 35 = 1295 troubled cells against at most 1024 workgroups."""
    wl = W.vortex(37, N)
    wl.ncell = (37, 35)
    o, g = paired_mixed(wl, m=0, mask=np.ones(wl.num_cells, dtype=np.uint8))
    worst, steps = run_mixed(o, g, 2)
    assert steps == 2 and worst > 0
    assert o.troubled().all() and g.troubled().all()


@pytest.mark.parametrize("form", ["fp64", "mixed"])
def test_3d_degree_9(form):
    wl = W.contact_wave(3, 9, 3)
    wl.ncell = (3, 2, 2)
    mask = W.random_mask(wl.num_cells, 0.5, seed=9)
    assert 0 < mask.sum() < wl.num_cells
    if form == "fp64":
        o, g = paired(wl, m=0, mask=mask)
        run_parity(o, g, 2, tol_init=1e-12)
    else:
        o, g = paired_mixed(wl, m=0, mask=mask)
        worst, steps = run_mixed(o, g, 2)
        assert steps == 2 and worst > 0
    assert o.troubled()[mask.astype(bool)].all()
