"""The far-wing test at segment lengths beyond FP32's range, against the oracle: models whose
lengths are scaled down and densities up by the same factor have the same optical depths, so
the segments that may be crossed in one step are the same.  The flow carries cells up to 8
widths off the quadrature, where many have opacity enough to count.  FP64 agrees to 1e-10 as
everywhere."""
import numpy as np
import pytest

from synth import configs, directions

from _common import oracle_for, rel, solver_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exponent", [0, 130, 260])
@pytest.mark.parametrize("long_segments", [0, 1])
def test_far_segments_of_any_length(exponent, long_segments):
    w = configs.outflow5(n_points=300, seed=5, nside=1)
    w.quad_x, w.quad_w = directions.uniform_grid(31, 4.0)
    w.model.vel *= 0.08
    w.model.pos *= 2.0 ** -exponent          # the scaling is exact
    w.model.n_h2 *= 2.0 ** exponent
    o = oracle_for(w)
    pops = o.lte()
    ref = o.formal_solve(pops)
    s = solver_for(w, long_segments=long_segments)
    for g, r in zip(s.formal_solve(pops), ref):
        assert np.isfinite(g).all() and rel(g, r).max() <= 1e-10
