"""Scattering where the line's source function is many orders above the mean intensity: a
background in the Wien regime (or no mean intensity yet at all) seen through gas whose scattering
opacity is a thousand times the line's, on one side of the cloud without any line opacity.  What
light there is comes from the line's small share of the emission, so nothing of the size of S
times a rounding may enter.  Isotropic and with a dipole, even and uneven quadratures; J and L*
against the oracle to 1e-9 as the other scattering tests, J_nu to 1e-9 of its largest value at the
point (offsets on the dark side of a line are differences of two intensities)."""
import numpy as np
import pytest

from synth import configs, directions

from _common import oracle_for, rel, solver_for

pytestmark = pytest.mark.gpu


def check(t_cmb, grid, dipole, dark):
    w = configs.outflow5(n_points=150, seed=17, nside=1)
    w.t_cmb = t_cmb
    w.quad_x, w.quad_w = directions.uniform_grid(15, 3.0) if grid == "uniform" else directions.gauss_hermite(12)
    m = w.model
    m.vel *= 0.4
    m.abundance[m.pos[:, 0] > 0.0] = 0.0
    o = oracle_for(w)
    pops = o.lte()
    nl, nq = w.species.n_lines, len(w.quad_x)
    kap = np.max([o.pair_nodes(pops, p, 0)["kappa"].max(axis=0) for p in range(0, 150, 15)], axis=0)
    chi = 1e3 * kap[None, :] * np.random.default_rng(2).uniform(0.5, 2.0, (150, nl))
    dip = 0.2 * chi[:, :, None] * np.array([0.6, 0.0, 0.8]) if dipole else None
    jnu = np.zeros((150, nl, nq)) if dark else o.scattering_start()
    s = solver_for(w)
    s.set_scattering(chi)
    if dipole:
        s.set_scattering_dipole(dip)
    J, _, L, Jn = s.formal_solve_scat(pops, jnu)
    rJ, _, rL, rJn = o.formal_solve_scat(pops, chi, jnu, chi_dip=dip)
    assert rel(J, rJ).max() <= 1e-9 and rel(L, rL).max() <= 1e-9
    assert (np.abs(Jn - rJn) / np.abs(rJn).max(axis=2, keepdims=True)).max() <= 1e-9


@pytest.mark.parametrize("t_cmb", [0.5, 2.725])
@pytest.mark.parametrize("grid", ["uniform", "hermite"])
@pytest.mark.parametrize("dipole", [False, True])
@pytest.mark.parametrize("dark", [False, True])
def test_weak_background(t_cmb, grid, dipole, dark):
    check(t_cmb, grid, dipole, dark)


@pytest.mark.parametrize("grid", ["uniform", "hermite"])
@pytest.mark.parametrize("dipole", [False, True])
def test_far_wings_light_dark_gas(grid, dipole):
    """S / J from 2^79 to 2^318: the far wings, 2^-75 of the scattering opacity and less, are the
    only light of the gas without line opacity."""
    check(0.1, grid, dipole, False)
