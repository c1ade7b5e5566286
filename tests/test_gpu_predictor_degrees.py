"""The FP32 predictor at every degree built, in the plain mixed form and the deviation form, against
the FP64 oracle: the matrix unit's row groups hold 4 of an operator's n rows, so every degree pads
them differently (n = 4 and 8: not at all; n = 5 and 9: 3 of 4 rows of the last group), the even /
odd form of the derivative starts at n = 6, and a workgroup holds another number of cells at every
degree.  Grids of odd extents leave the last workgroup partly filled; one cell leaves it almost
empty.  Unlimited steps: every value of the new state comes from the predictor.

Tolerance of the other mixed-precision tests: 2e-6 of each variable's scale per step.
"""
import pytest

from paper_1406_7416_amd import workloads as W
from test_gpu_mixed import paired_mixed, run_mixed
from test_gpu_mixed_dev import paired_dev

pytestmark = pytest.mark.gpu

CASES = [(2, N) for N in range(1, 10)] + [(3, 1), (3, 2), (3, 3), (3, 9)]


@pytest.mark.parametrize("pair", [paired_mixed, paired_dev])
@pytest.mark.parametrize("dim,N", CASES)
def test_unlimited_steps(dim, N, pair):
    wl = W.contact_wave(dim, N, 3)
    wl.ncell = (7, 5) if dim == 2 else ((3, 2, 1) if N == 9 else (3, 5, 3))
    o, g = pair(wl, m=0, detect=False)
    worst, steps = run_mixed(o, g, 2)
    assert steps == 2 and worst > 0


@pytest.mark.parametrize("pair", [paired_mixed, paired_dev])
@pytest.mark.parametrize("N", [3, 9])
def test_one_cell(N, pair):
    wl = W.vortex(1, N)
    o, g = pair(wl, m=0, detect=False)
    run_mixed(o, g, 2)
