"""The space-time predictor at every degree built and in every form with the limiter off, against the FP64
oracle without limiter: nothing overwrites a cell after the predictor, the faces and the corrector, so that
wrong values of any node reach the comparison.  Grids of odd extents leave the last workgroup partly filled;
one cell leaves it almost empty (idle lanes, the tail of the line order, the last cell's bounds).

Tolerances of the other parity tests: FP64 1e-12 of each variable's scale on the first step, 1e-10 after;
mixed and deviation forms 2e-6 per step.
"""
import pytest

from oracle import oracle as O
from paper_1406_7416_amd import workloads as W
from test_gpu_parity import gpu_problem, rel_err

pytestmark = pytest.mark.gpu

CASES = [(2, N) for N in range(1, 10)] + [(3, 1), (3, 2), (3, 3), (3, 9)]
FORMS = {"fp64": (0, (1e-12, 1e-10)), "mixed": (1, (2e-6, 2e-6)), "dev": (2, (2e-6, 2e-6))}


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("one_cell", [False, True])
@pytest.mark.parametrize("dim,N", CASES)
def test_two_steps(dim, N, one_cell, form):
    wl = W.contact_wave(dim, N, 3)
    wl.ncell = (1,) * dim if one_cell else (7, 5) if dim == 2 else (3, 2, 1) if N == 9 else (3, 5, 3)
    precision, tol = FORMS[form]
    o = O.Oracle(wl, limiter=False)
    u, _ = o.project(wl.ic, 0)
    o.set_state(u, None)
    g = gpu_problem(wl, precision=precision, limiter=False)
    g.set_state(u, None)
    errors = []
    for bound in tol:
        dt = o.cfl_dt()
        o.step(dt)
        g.step(dt)
        errors.append(rel_err(g.state(), o.state()))
        assert errors[-1] < bound, errors
    assert precision == 0 or max(errors) > 1e-12   # the reduced forms are at work
    assert g.troubled().sum() == 0 and o.troubled().sum() == 0
