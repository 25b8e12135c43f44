"""The rate equations at every number of levels (the matrices of 2 to 11 are solved from
registers, 12 and more from private memory) and at point counts around a wave's 64, against
the oracle's: random lines and collision pairs in any order, some pairs twice, rates on both
sides of the conservation row's 1 so that rows change places, and points whose solution with
the ALO, or altogether, is rejected.

Rates over eight decades in random order make ill-conditioned systems, whose solutions
follow the last bit of every exponential (register and private-memory eliminations agree
bit for bit, and both differ from the oracle by up to 1e-6 of a population).  So the flags
are compared with the oracle's and the populations put back into the equations: partial
pivoting leaves a residual of at most about 3 n^2 eps (1e-13 for 16 levels) times the largest
row sum, the largest population and the elimination's growth, here taken as ten.  Tame
systems are compared population by population in the parity tests."""
import numpy as np
import pytest

from synth import directions, species
from synth.configs import Workload
from synth.models import power_law_sphere

from _common import oracle_for, solver_for

pytestmark = pytest.mark.gpu

H, KB, C = 6.62607015e-27, 1.380649e-16, 2.99792458e10


def random_species(n, rng):
    E = np.sort(rng.uniform(0.0, 300.0, n)) * 1.38e-16
    E[0] = 0.0
    pairs = [(u, l) for u in range(n) for l in range(u) if E[u] > E[l]]
    lines = [(u, u - 1) for u in range(1, n)] + [pairs[i] for i in rng.permutation(len(pairs))[: min(5, len(pairs))]]
    rng.shuffle(lines)
    coll = pairs + [pairs[i] for i in rng.permutation(len(pairs))[: len(pairs) // 3]]
    coll = [(b, a) if rng.random() < 0.2 else (a, b) for a, b in coll]   # table entries either way round
    rng.shuffle(coll)
    T = np.geomspace(5.0, 500.0, 7)
    return species.Species(energy=E, weight=rng.integers(1, 9, n).astype(float), mass=28 * species.AMU,
                           line_up=np.array([p[0] for p in lines], np.int32), line_lo=np.array([p[1] for p in lines], np.int32),
                           line_A=10.0 ** rng.uniform(-6, 2, len(lines)), coll_up=np.array([p[0] for p in coll], np.int32),
                           coll_lo=np.array([p[1] for p in coll], np.int32), coll_T=T,
                           coll_K=1e-10 * rng.uniform(0.2, 5.0, (len(coll), 7)))


@pytest.mark.parametrize("n_lev", range(2, 17))
@pytest.mark.parametrize("points", [13, 64, 129])
def test_rates_at_every_level_count(n_lev, points):
    rng = np.random.default_rng([n_lev, points])
    m = power_law_sphere(3, points, 1e17, 1e15, 1e6, -1.0, 60.0, -0.4, 0.0, 1e-6)
    m.temperature[:4] = [1.0, 5.0, 500.0, 2000.0]   # the table's ends and beyond them
    x, wq = directions.uniform_grid(31)
    w = Workload("rates", m, random_species(n_lev, rng), directions.axis_pair(), x, wq)
    s, o = solver_for(w, trace=False), oracle_for(w)
    nl = w.species.n_lines
    old = o.lte()
    J = 10.0 ** rng.uniform(-16, -10, (points, nl))
    L = rng.uniform(0.0, 0.95, (points, nl))
    Je = J * rng.uniform(0.2, 1.0, (points, nl))
    Je[5], J[7], Je[7] = np.nan, np.nan, np.nan      # flags 1 and 2
    got, flags = s.stateq(old, J, Je, L)
    _, ref_flags = o.stateq(old, J, Je, L)
    assert np.array_equal(flags, ref_flags) and flags[5] == 1 and flags[7] == 2
    assert np.array_equal(got[7], old[7])
    sp = w.species
    nu = (sp.energy[sp.line_up] - sp.energy[sp.line_lo]) / H
    Bul = sp.line_A * C * C / (2 * H * nu ** 3)
    M = np.zeros((points, n_lev, n_lev))

    def rate(a, b, R):
        M[:, b, a] += R
        M[:, a, a] -= R

    alo = flags == 0
    F, Ls = np.where(alo[:, None], Je, J), np.where(alo[:, None], L, 0.0)
    for l, (u, lo) in enumerate(zip(sp.line_up, sp.line_lo)):
        rate(u, lo, sp.line_A[l] * (1 - Ls[:, l]) + Bul[l] * F[:, l])
        rate(lo, u, Bul[l] * sp.weight[u] / sp.weight[lo] * F[:, l])
    T = m.temperature
    for c, (u, lo) in enumerate(zip(sp.coll_up, sp.coll_lo)):
        K = np.interp(T, sp.coll_T, sp.coll_K[c]) * m.n_h2
        rate(u, lo, K)
        rate(lo, u, K * sp.weight[u] / sp.weight[lo] * np.exp(-(sp.energy[u] - sp.energy[lo]) / (KB * T)))
    M[:, 0, :] = 1.0
    b = np.zeros((points, n_lev))
    b[:, 0] = m.abundance * m.n_h2
    solved = flags < 2
    assert solved.sum() >= points - points // 4
    res = np.abs((M @ got[:, :, None])[:, :, 0] - b).max(axis=1)
    bound = 1e-12 * np.abs(M).sum(axis=2).max(axis=1) * got.max(axis=1)
    assert (res[solved] <= bound[solved]).all()
