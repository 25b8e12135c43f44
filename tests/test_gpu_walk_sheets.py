"""Walks through points in sheets across the rays: neighbours in the same sheet lie ahead or
behind by 0 to 1e-6 of their distance, which the FP32 evaluation cannot tell, and some of them
are nearest to the line, some rival the best and most do not matter; against the oracle's FP64
walk, cell by cell."""
import numpy as np
import pytest

from synth import directions, species
from synth.configs import Workload
from synth.models import knn, power_law_sphere

from _common import oracle_for, solver_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wobble", [0.0, 1e-12, 1e-9, 1e-7, 1e-6])
@pytest.mark.parametrize("axis", [0, 2])
def test_sheets(wobble, axis):
    rng = np.random.default_rng([7, axis])
    n, sheets = 900, 9
    m = power_law_sphere(7, n, 1e17, 1e15, 1e5, -2.0, 30.0, 0.0, 5e5, 1e-8)
    h = 2e17 / sheets
    m.pos[:, axis] = (rng.integers(0, sheets, n) - sheets // 2) * h + wobble * h * rng.standard_normal(n)
    m.nbr = knn(m.pos, 16)
    one = np.zeros(3)
    one[axis] = 1.0
    rays = np.array([one, -one])
    x, wq = directions.uniform_grid(31)
    w = Workload("sheets", m, species.two_level(), rays, x, wq)
    s, o = solver_for(w), oracle_for(w)
    off, cells = o.walk_all()
    assert s.trace_stats()[0] == off[-1] and off[-1] > 2 * n
    for q in range(2 * n):
        assert np.array_equal(s.get_ray(q // 2, q % 2), cells[off[q]:off[q + 1]]), q
