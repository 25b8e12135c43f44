"""Very opaque velocity sub-steps against the oracle: every step multiplies the elimination
state by the square of its optical depth (here up to 2^68), so the state passes the rescaling
threshold within a few steps, wherever the sweep is: in runs of cells without sub-steps, at
their boundary with a segment that has some, on either side of an exact restart of the
profile's recurrence with every remainder modulo four before it, and at staging rounds of two
nodes and of many.  One, two, three and five lines per lane, both segment modes, both
precisions.  J and L* agree to 1e-10 as everywhere, FP32 to its own 1e-4.  Jeff, down to 1e-46
of J here, is compared with the oracle's on the scale of J (the oracle's carries the rounding of
a difference), and between the FP64 forms, which add and multiply positive numbers only, for
itself."""
import numpy as np
import pytest

from synth import directions, species
from synth.configs import Workload
from synth.models import chain_1d

from _common import oracle_for, rel, solver_for

pytestmark = pytest.mark.gpu

F_SUB = 0.5


def _workload(n_lev, seed, peak):
    """A chain whose neighbours move by 0 to 30 widths against each other, with the distance
    between two of them growing with the number of sub-steps: every step's optical depth at the
    line's centre is up to 2^peak."""
    rng = np.random.default_rng([n_lev, seed])
    n = 70
    sp = species.linear_rotor(n_lev)
    T = 20.0
    width = np.sqrt(2 * 1.380649e-16 * T / sp.mass + 1.5e4 ** 2)
    dv = np.where(rng.random(n - 1) < 0.4, rng.uniform(0.0, 0.9 * F_SUB, n - 1), rng.uniform(0.5, 30.0, n - 1))
    dv *= np.where(rng.random(n - 1) < 0.5, -1.0, 1.0)
    v = np.concatenate([[0.0], np.cumsum(dv)]) * width
    m = np.maximum(1.0, np.ceil(np.abs(dv) / F_SUB))
    x = np.concatenate([[0.0], np.cumsum(1e15 * m * rng.uniform(0.25, 1.0, n - 1))])
    model = chain_1d(x, v, 1e5, T, 1.5e4, 1e-8)
    q, wq = directions.uniform_grid(31)
    w = Workload("opaque", model, sp, directions.axis_pair(), q, wq, f_sub=F_SUB)
    o = oracle_for(w)
    kap = max(o.pair_nodes(o.lte(), n // 2, 0)["kappa"].max(axis=0))
    model.abundance *= 2.0 ** peak / (kap * 1e15)
    return w


@pytest.mark.parametrize("lpl, n_lev", [(1, 2), (2, 5), (3, 6), (5, 10)])
@pytest.mark.parametrize("peak", [40, 68])
def test_opaque_steps_match_the_oracle(lpl, n_lev, peak):
    for seed in range(4):
        w = _workload(n_lev, seed, peak)
        o = oracle_for(w)
        pops = o.lte() * np.random.default_rng(seed).uniform(0.97, 1.03, (w.n_points, n_lev))
        rJ, rE, rL = o.formal_solve(pops)
        s = solver_for(w)
        first = None
        for prec, tol in (("fp64", 1e-10), ("fp32", 1e-4)):
            for kw in (dict(long_segments=0), dict(long_segments=1), dict(long_segments=1, stage_nodes=2)):
                s.set_params(precision=prec, **{"stage_nodes": 0, "lines_per_lane": lpl, **kw})
                assert s.launch()["lines_per_lane"] == lpl
                J, E, L = s.formal_solve(pops)
                assert np.isfinite(J).all() and np.isfinite(E).all() and np.isfinite(L).all(), (seed, prec, kw)
                assert rel(J, rJ).max() <= tol and rel(L, rL).max() <= tol, (seed, prec, kw)
                assert (np.abs(E - rE) / rJ).max() <= tol, (seed, prec, kw)
                if prec == "fp64":
                    first = E if first is None else first
                    assert rel(E, first).max() <= tol, (seed, kw)
