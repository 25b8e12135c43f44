"""The coupled solve of the band operator on the device: every number of levels it keeps in
registers at its ends (2, 5, 11) and the general form (12, 16) against a sparse LU; blocks
of four waves and blocks that take several groups of points (many copies of a model, which do
not couple, give each copy what the single model gets); more steps than are enqueued at once,
and a solve with nothing to couple.

The solve stops at a residual of 1e-13 of the norm of x, both in fractional populations, so
an element may be off by 1e-13 sqrt(P) ||A^-1|| of its point's density; the bound takes 100 for
the last factor.  (Populations far below their point's density have no relative accuracy.)"""
import numpy as np
import pytest

from oracle import band
from synth import configs, directions, species
from synth.models import concat_models

from _common import oracle_for, solver_for

pytestmark = pytest.mark.gpu


def _agree(got, ref, w):
    nt = (w.model.abundance * w.model.n_h2)[:, None]
    err = (np.abs(got - ref) / nt).max()
    print("error %.1e" % err)
    return err <= 1e-11 * np.sqrt(w.n_points)


def _case(levels, points=200, seed=3):
    w = configs.outflow5(n_points=points, seed=seed, nside=1)
    w.model.temperature = w.model.temperature + 1000.0  # (no population so small that its sign is rounding)
    w.species = species.linear_rotor(levels) if levels > 2 else species.two_level()
    return w


@pytest.mark.parametrize("levels", [2, 5, 11, 12, 16])
def test_levels_match_sparse_lu(levels):
    w = _case(levels)
    o = oracle_for(w)
    pops = o.lte() * np.random.default_rng(levels).uniform(0.9, 1.1, (w.n_points, levels))
    args = o.formal_solve_band(pops)
    ref, ok = band.stateq_band(o, pops, *args, band.first_cells(o))
    got, used, its = solver_for(w).stateq_band(pops, *args)
    assert bool(used) == bool(ok)
    assert _agree(got, ref, w)


@pytest.mark.parametrize("copies", [43, 173])   # 17,200 points: four waves a block; 69,200: two rounds
def test_copies_of_a_model(copies):
    w = configs.sphere2(n_points=400, seed=4)
    w.model.abundance[:] = 1e-6
    o = oracle_for(w)
    pops = o.lte() * np.random.default_rng(1).uniform(0.9, 1.1, (400, 2))
    s = solver_for(w)
    args = s.formal_solve_band(pops)
    ref, used, _ = s.stateq_band(pops, *args)
    assert used
    offs, m = concat_models([w.model] * copies)
    many = configs.Workload("copies", m, w.species, w.rays, w.quad_x, w.quad_w, offsets=offs)
    rep = lambda a: np.concatenate([a] * copies)
    got, used, its = solver_for(many).stateq_band(rep(pops), *(rep(a) for a in args))
    assert used == copies
    assert _agree(got, rep(ref), many)


def test_many_steps_and_none():
    # opaque cells and neighbours that count several times couple strongly: 6 to 40 steps, the
    # last with populations that are not positive, where both take the local solve
    most = 0
    for abundance, scale in ((1e-5, 10), (2e-5, 8), (3e-5, 6), (1e-4, 20), (1e-5, 0)):
        w = configs.sphere2(n_points=400, seed=4)
        w.model.abundance[:] = abundance
        o = oracle_for(w)
        pops = o.lte()
        s = solver_for(w)
        J, Je, L, Jb, Ld, Ln = s.formal_solve_band(pops)
        ref, ok = band.stateq_band(o, pops, J, Je, L, Jb, Ld, scale * Ln, band.first_cells(o))
        got, used, its = s.stateq_band(pops, J, Je, L, Jb, Ld, scale * Ln)
        print("steps", its, used, ok)
        assert bool(used) == bool(ok)
        assert _agree(got, ref, w)
        assert (its == 0) == (scale == 0)
        most = max(most, its)
    assert most > 10


@pytest.mark.parametrize("points, n_q, levels, lpl", [(2, 31, 2, 0), (65, 31, 5, 1), (130, 100, 5, 2), (300, 33, 12, 2)])
def test_split_pairs_of_the_band(points, n_q, levels, lpl):
    # few points: each pair of rays on a wave of its own; against the oracle
    w = _case(levels, points, seed=points)
    w.quad_x, w.quad_w = directions.uniform_grid(n_q, 4.0)
    o = oracle_for(w)
    pops = o.lte()
    got, ref = solver_for(w, lines_per_lane=lpl).formal_solve_band(pops), o.formal_solve_band(pops)
    for g, r in zip(got[:5], ref[:5]):   # (Jb is Jeff less the band's share: on the scale of Jeff)
        assert (np.abs(g - r) / np.maximum(np.abs(ref[1] if r is ref[3] else r), 1e-300)).max() <= 1e-10
    scale = np.maximum(np.abs(ref[5]).max(axis=2, keepdims=True), 1e-300)
    assert (np.abs(got[5] - ref[5]) / scale).max() <= 1e-10
