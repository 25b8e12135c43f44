"""The Boltzmann factors of the collision rates to the last bits: two levels without radiation,
whose excited fraction is C_lu / (C_ul + C_lu) = q / (1 + q), q = g_u/g_l e^{-E/kT}.

Tolerance, in half ulps (1.1e-16) of the fraction: on the GPU the exponential 2, its two products
2, the sum 1, the elimination's product and quotient 2; in numpy the exponential 2, the product,
the sum and the quotient 3, the fraction of the density 1; the argument is the same quotient of
the same two numbers on both sides.  13 in all: 1.5e-15.

Temperatures go down to where 1/kT leaves the FP64 range: levels of equal energy keep the ratio
of their statistical weights there (residual of a 3 x 3 elimination: 1e-14)."""
import numpy as np
import pytest

from synth import directions, species
from synth.configs import Workload
from synth.models import power_law_sphere

from _common import solver_for

pytestmark = pytest.mark.gpu

KB = 1.380649e-16


def _solve(E, g, A, coll, T, J):
    n = len(T)
    m = power_law_sphere(3, n, 1e17, 1e15, 1e6, 0.0, 60.0, 0.0, 0.0, 1e-6)
    m.temperature[:] = T
    sp = species.Species(energy=np.array(E), weight=np.array(g), mass=28 * species.AMU,
                         line_up=np.array([len(E) - 1], np.int32), line_lo=np.array([0], np.int32),
                         line_A=np.array([A]), coll_up=np.array([c[0] for c in coll], np.int32),
                         coll_lo=np.array([c[1] for c in coll], np.int32), coll_T=np.array([1.0, 1e4]),
                         coll_K=np.full((len(coll), 2), 1e-10))
    x, wq = directions.uniform_grid(31)
    s = solver_for(Workload("boltzmann", m, sp, directions.axis_pair(), x, wq), trace=False)
    nt = m.abundance * m.n_h2
    field = np.full((n, 1), J)
    pops, flags = s.stateq(np.repeat(nt[:, None] / len(E), len(E), axis=1), field, field, np.zeros((n, 1)))
    assert (flags == 0).all()
    return pops / nt[:, None]


@pytest.mark.parametrize("g", [0.5, 1.0, 3.0])
def test_excited_fraction(g):
    E = 4e-15
    T = E / KB / np.linspace(0.0, 5.0, 4001)[1:]
    got = _solve([0.0, E], [1.0, g], 0.0, [(1, 0)], T, 0.0)[:, 1]
    q = g * np.exp(-E / (KB * T))
    assert np.abs(got / (q / (1.0 + q)) - 1.0).max() <= 1.5e-15


@pytest.mark.parametrize("n_lev", [3, 13])   # from registers and from private memory
def test_levels_of_equal_energy_at_any_temperature(n_lev):
    T = np.array([1e-300, 1e-295, 1e-280, 1e-100, 1.0, 100.0])
    E = [0.0] * (n_lev - 1) + [4e-16]
    g = [1.0 + i for i in range(n_lev)]
    got = _solve(E, g, 1e-5, [(i, 0) for i in range(1, n_lev - 1)], T, 1e-13)
    for i in range(1, n_lev - 1):
        assert np.abs(got[:, i] / got[:, 0] / g[i] - 1.0).max() <= 1e-14
