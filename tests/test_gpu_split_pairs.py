"""A point's ray pairs split over several waves (few points) against one wave per point (the
grid launch, which never splits): the per-pair sums are added in the same order, so the
results agree bit for bit; and against the oracle.  One point to one workgroup's worth, one
pair to many, frequencies in chunks, several waves per point's lines, FP32 and FP64, and
models already converged, whose points keep what they hold."""
import numpy as np
import pytest

from synth import configs, directions, species

from _common import oracle_for, rel, solver_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("points, nside, n_q, levels", [(2, 0, 31, 5), (13, 1, 31, 2), (65, 1, 100, 5), (130, 2, 31, 16),
                                                       (700, 2, 33, 10), (300, 3, 7, 5)])
def test_split_pairs_bitwise(points, nside, n_q, levels):
    import torch
    w = configs.outflow5(n_points=points, seed=points, nside=max(nside, 1))
    if nside == 0:
        w.rays = directions.axis_pair()
    w.species = species.linear_rotor(levels)
    w.quad_x, w.quad_w = directions.uniform_grid(n_q, 4.0)
    s, o = solver_for(w), oracle_for(w)
    pops = o.lte()
    ref = o.formal_solve(pops)
    dp = torch.tensor(pops, device="cuda:0")
    for prec, tol in (("fp64", 1e-10), ("fp32", 1e-4)):
        got = []
        for persistent in (0, 1):
            s.set_params(precision=prec, persistent=persistent)
            out = [torch.full((points, levels - 1), np.nan, dtype=torch.float64, device="cuda:0") for _ in range(3)]
            s.formal_solve_dev(dp, *out)
            torch.cuda.synchronize()
            got.append([t.cpu().numpy() for t in out])
        for a, b, r in zip(*got, ref):
            assert np.array_equal(a, b), prec
            assert rel(a, r).max() <= tol, prec


def test_split_pairs_with_converged_models():
    """An ALI over models of very different opacity: the thin ones stop first."""
    from synth.models import concat_models, power_law_sphere
    ms = [power_law_sphere(30 + i, 150, 1e17, 1e15, 10.0 ** (3 + i), -2.0, 30.0, 0.0, 2e5, 10.0 ** (-9 + i)) for i in range(3)]
    offs, m = concat_models(ms)
    x, wq = directions.uniform_grid(31)
    w = configs.Workload("three", m, species.two_level(), directions.healpix_ring(1), x, wq, offsets=offs, max_iter=60)
    out = []
    for persistent in (0, 1):
        s = solver_for(w, persistent=persistent, tol=1e-8)
        pops, rep = s.run_ali()
        out.append((pops, s.model_status()))
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1][0], out[1][1][0]) and len(set(out[0][1][0])) > 1
