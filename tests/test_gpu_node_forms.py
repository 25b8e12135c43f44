"""The two ways in which the formal solve reads a staged node (a lane's own value broadcast
over its row of 16 lanes, or every value by every lane) and its segments taken singly or in
pairs: staging windows of two to six nodes cut runs of segments without sub-steps, runs of
far-wing segments and segments with sub-steps at every place, for each number of lines per
lane.  The cuts change no arithmetic, so a mode's results agree bit for bit; all agree with
the oracle."""
import numpy as np
import pytest

from synth import configs, species

from _common import oracle_for, rel, solver_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision, tol", [("fp64", 1e-10), ("fp32", 1e-4)])
@pytest.mark.parametrize("slow", [0.03, 0.3])
def test_staging_windows_bitwise(precision, tol, slow):
    import torch
    w = configs.outflow5(n_points=400, seed=9, nside=1)
    w.model.vel = w.model.vel * slow
    w.species = species.linear_rotor(10)
    s, o = solver_for(w, precision=precision), oracle_for(w)
    pops = o.lte()
    ref = o.formal_solve(pops)
    dp = torch.tensor(pops, device="cuda:0")
    for long_mode in (0, 1):
        first = None
        for lpl in (1, 2, 3, 4, 5):
            for nodes in (0, 2, 3, 4, 5, 6):
                s.set_params(precision=precision, lines_per_lane=lpl, long_segments=long_mode, stage_nodes=nodes)
                out = [torch.full((w.n_points, 9), np.nan, dtype=torch.float64, device="cuda:0") for _ in range(3)]
                s.formal_solve_dev(dp, *out)
                torch.cuda.synchronize()
                got = [t.cpu().numpy() for t in out]
                if first is None:
                    first = got
                    assert all(rel(g, r).max() <= tol for g, r in zip(got, ref))
                assert all(np.array_equal(g, f) for g, f in zip(got, first)), (long_mode, lpl, nodes)
