"""The ray walk's FP32 evaluation against the oracle's FP64 walk, cell by cell, where the two
could part: lattices whose neighbours lie across or symmetric about axis rays, points that
coincide or sit nearer than FP32 can tell at the model's scale, clouds far from the origin
of the coordinates or on scales beyond FP32's range, neighbour lists with unused slots and
of every length modulo four, and point counts around a workgroup's 64."""
import numpy as np
import pytest

from synth import configs, directions, species
from synth.configs import Workload
from synth.models import lattice_3d, power_law_sphere

from _common import oracle_for, solver_for

pytestmark = pytest.mark.gpu


def cloud(n, k=12, scale=1e17, shift=0.0, seed=5):
    m = power_law_sphere(seed, n, scale, 0.01 * scale, 1e5, -2.0, 30.0, 0.0, 5e5, 1e-8, k=k)
    m.pos += shift
    return m


def pairs_of_near_points(n, gap):
    """Every second point sits `gap` extents from its predecessor."""
    m = cloud(n, k=9)
    m.pos[1::2] = m.pos[0::2] + gap * 2e17
    return m


def ragged(n):
    m = cloud(n, k=13)
    m.nbr[::3, 4:] = -1
    m.nbr[1::3, :5] = -1
    m.nbr[::17, :] = -1
    return m


def flat(m):
    m.pos[:, 2] = 0.0
    return m


CASES = {
    "lattice": (lambda: lattice_3d(7, 1e15), 1),
    "lattice, every neighbour tied": (lambda: lattice_3d(6, 1e15), 2),
    "coincident": (lambda: pairs_of_near_points(200, 0.0), 1),
    "below FP32 at this scale": (lambda: pairs_of_near_points(200, 1e-12), 1),
    "at the bound": (lambda: pairs_of_near_points(200, 1.0001e-8), 1),
    "far from the origin": (lambda: cloud(300, shift=1e23), 2),
    "beyond FP32's range": (lambda: cloud(300, scale=1e60), 1),
    "below FP32's range": (lambda: cloud(300, scale=1e-60), 1),
    "ragged": (lambda: ragged(500), 2),
    "flat": (lambda: flat(cloud(300)), 2),
    "63 points": (lambda: cloud(63, k=5), 1),
    "64 points": (lambda: cloud(64, k=6), 1),
    "65 points": (lambda: cloud(65, k=7), 1),
    "one point": (lambda: cloud(1, k=1), 1),
}


@pytest.mark.parametrize("name", CASES)
def test_walk_equals_the_oracle(name):
    make, nside = CASES[name]
    m = make()
    if name == "one point":
        m.nbr[:] = -1
    x, wq = directions.uniform_grid(31)
    rays = directions.axis_pair() if name == "lattice" else directions.healpix_ring(nside)
    w = Workload("walk", m, species.two_level(), rays, x, wq)
    s, o = solver_for(w), oracle_for(w)
    off, cells = o.walk_all()
    n = m.n_points * rays.shape[0]
    assert s.trace_stats()[0] == off[-1] and s.trace_stats()[1] == np.diff(off).max()
    for q in range(0, n, max(1, n // 1500)):
        assert np.array_equal(s.get_ray(q // rays.shape[0], q % rays.shape[0]), cells[off[q]:off[q + 1]]), q


@pytest.mark.parametrize("n", [100, 1000])
def test_costs_and_steps_follow_the_walks(n):
    """Per point: one per ray plus, per segment outward, the sub-steps of the sweep's rule."""
    w = configs.outflow5(n_points=n, seed=13, nside=1)
    s, o = solver_for(w), oracle_for(w)
    off, cells = o.walk_all()
    vw, m, R = o.line_width_speed(), w.model, w.rays.shape[0]
    cost = np.zeros(n, np.int64)
    for q in range(n * R):
        O, r = divmod(q, R)
        c = np.concatenate([[O], cells[off[q]:off[q + 1]]])
        d = m.vel[c] - m.vel[O]
        u = w.rays[r]
        sv = (d[:, 0] * u[0] + d[:, 1] * u[1]) + d[:, 2] * u[2]
        ds, thr = np.abs(np.diff(sv)), w.f_sub * np.minimum(vw[c[1:]], vw[c[:-1]])
        cost[O] += 1 + int(np.where(ds > thr, np.ceil(ds / thr), 1).sum())
    assert np.array_equal(s.point_cost(), cost)
    assert s.trace_stats()[2] == cost.sum() - n * R
    order = s.order()
    assert np.array_equal(np.sort(order), np.arange(n))
