"""The mixed form at the edge of FP32's range: one node's density beyond it (1e39: infinite in the FP32
working precision, finite in the FP64 state).  Momentum and energy do not see it: the velocity there is
zero, so their fluxes are finite, and every value of theirs stays the one of the FP64 form.

Tolerance of the other mixed-precision tests: 2e-6 of each variable's scale per step.
"""
import numpy as np
import pytest

from paper_1406_7416_amd import workloads as W
from test_gpu_parity import gpu_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,N", [(2, 1), (2, 3), (2, 5), (2, 9), (3, 2), (3, 3)])
def test_infinite_density_leaves_momentum_and_energy(dim, N):
    from paper_1406_7416_amd import adg
    wl = W.contact_wave(dim, N, 3)
    n = N + 1
    out = []
    for precision in (adg.ADG_FP64, adg.ADG_MIXED):
        g = gpu_problem(wl, precision=precision, limiter=False)
        u, _ = g.project(wl.ic, 0)
        u[0, wl.num_cells // 2, sum(n ** k for k in range(dim))] = 1e39   # node (1, 1(, 1)) of the middle cell
        g.set_state(u)
        g.step(1e-3)
        out.append(g.state()[1:])
    exact, mixed = out
    assert np.isfinite(exact).all()
    assert np.isfinite(mixed).all(), f"{np.count_nonzero(~np.isfinite(mixed))} values"
    for v in range(dim + 1):
        assert np.abs(mixed[v] - exact[v]).max() < 2e-6 * np.abs(exact[v]).max()
