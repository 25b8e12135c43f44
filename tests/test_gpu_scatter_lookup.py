"""Scattering on quadratures whose offsets are uneven in every way the lookup table meets (an
offset or none per bin, many in one bin, one offset, 256) and with scattering from far
below to far above the line's opacity, which decides where the line counts no more; against
the oracle."""
import numpy as np
import pytest

from synth import configs

from _common import oracle_for, rel, solver_for

pytestmark = pytest.mark.gpu


def _grid(kind):
    if kind == "one":
        x = np.array([0.0])
    elif kind == "cluster":      # 9 offsets within a 256th of the range
        x = np.concatenate([np.linspace(0.0, 0.02, 5)[1:], [5.0]])
        x = np.concatenate([-x[::-1], [0.0], x])
    elif kind == "wide":         # ever farther apart
        x = 0.05 * 1.5 ** np.arange(12)
        x = np.concatenate([-x[::-1], x])
    elif kind == "many":
        x = np.sort(np.random.default_rng(3).uniform(0.01, 4.0, 128))
        x = np.concatenate([-x[::-1], x])
    w = np.exp(-x ** 2)
    return x, w / w.sum()


@pytest.mark.parametrize("kind, strength", [("one", 1.0), ("cluster", 1.0), ("wide", 1e-9), ("wide", 1e6), ("many", 1.0)])
def test_uneven_lookup(kind, strength):
    w = configs.outflow5(n_points=120, seed=6, nside=1)
    w.quad_x, w.quad_w = _grid(kind)
    o = oracle_for(w)
    rng = np.random.default_rng(8)
    pops = o.lte() * rng.uniform(0.8, 1.2, (w.n_points, w.species.n_lev))
    kap = np.median(o.pair_nodes(pops, 0, 0)["kappa"], axis=0)
    chi = strength * kap[None, :] * rng.uniform(0.5, 2.0, (w.n_points, w.species.n_lines))
    jnu = o.scattering_start() * rng.uniform(1.0, 4.0, (w.n_points, w.species.n_lines, len(w.quad_x)))
    s = solver_for(w)
    s.set_scattering(chi)
    J, Je, L, Jn = s.formal_solve_scat(pops, jnu)
    rJ, rJe, rL, rJn = o.formal_solve_scat(pops, chi, jnu)
    assert all(np.all(np.isfinite(a)) for a in (J, Je, L, Jn))
    assert rel(J, rJ).max() <= 1e-9 and rel(L, rL).max() <= 1e-9 and rel(Jn, rJn).max() <= 1e-9
    assert (np.abs(Je - rJe) / np.abs(rJ)).max() <= 1e-9
