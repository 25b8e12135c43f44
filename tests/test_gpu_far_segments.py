"""Far-wing segments eliminated in one step against the oracle, which steps through all of
them: where the bound on a segment's opacity is loose and where it is tight (the speed of
the flow against the width, the opacity of the cells), with a background far under the
gas's emission and one that is exactly zero (only segments whose opacity underflows may
then be skipped), one- and two-group lane maps, two-node staging windows and both segment
modes.  FP64 agrees to 1e-10 as everywhere; FP32's own tolerance is 1e-4."""
import numpy as np
import pytest

from synth import configs

from _common import oracle_for, rel, solver_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("speed, thick, t_cmb, n_q", [(0.1, 1.0, 2.725, 31), (1.0, 1.0, 2.725, 31), (6.0, 1.0, 2.725, 47),
                                                     (1.0, 1e5, 2.725, 31), (1.0, 1e-6, 2.725, 15), (1.0, 1.0, 0.2, 31),
                                                     (3.0, 1e3, 0.004, 31)])
def test_far_segments_match_the_oracle(speed, thick, t_cmb, n_q):
    w = configs.outflow5(n_points=400, seed=71, nside=1)
    w.model.vel *= speed
    w.model.abundance *= thick
    w.t_cmb = t_cmb
    from synth import directions
    w.quad_x, w.quad_w = directions.uniform_grid(n_q, 4.0)
    o = oracle_for(w)
    pops = o.lte()
    ref = o.formal_solve(pops)
    s = solver_for(w, profile=1)
    method = s.trace_stats()[2] * w.species.n_lines * n_q
    for prec, tol in (("fp64", 1e-10), ("fp32", 1e-4)):
        for kw in (dict(long_segments=0), dict(long_segments=1), dict(stage_nodes=2), dict(stage_nodes=64)):
            s.set_params(precision=prec, **{"long_segments": -1, "stage_nodes": 0, **kw})
            s.reset_kernel_stats()
            got = s.formal_solve(pops)
            if speed >= 1.0:
                assert 0 < s.executed_steps() < method
            for g, r in zip(got, ref):
                assert np.isfinite(g).all() and rel(g, r).max() <= tol, (prec, kw)
