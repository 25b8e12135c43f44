"""Images where the segments of a ray pair mix in every way the sweep treats apart: all without
sub-steps (taken two at a time, odd and even runs), a few sub-steps (evaluated directly),
many (the profile by recurrence), and very opaque cells, whose state has to be rescaled;
against the oracle."""
import numpy as np
import pytest

from synth import configs

from _common import oracle_for, rel, solver_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("speed, abundance", [(0.0, 1.0), (0.02, 1.0), (0.1, 1.0), (0.3, 1e8), (1.0, 1.0), (8.0, 1e6)])
def test_image_runs(speed, abundance):
    w = configs.outflow5(n_points=900, seed=12, nside=1)
    w.model.vel = w.model.vel * speed
    w.model.abundance = w.model.abundance * abundance
    s, o = solver_for(w), oracle_for(w)
    pops = s.lte()
    v = np.linspace(-1.0, 1.0, 67) * (1e5 + 1.2 * np.abs(w.model.vel).max())
    sel = np.random.default_rng(2).choice(w.n_points, 40, replace=False)
    for r in (0, 5):
        I, _ = s.image(pops, r, 1, v)
        Io, _ = o.image(pops, r, 1, v, points=sel)
        assert rel(I[sel], Io).max() <= 1e-10
        assert np.all(np.isfinite(I)) and np.all(I > 0)
