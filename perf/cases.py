"""What a program that uses the library has it do, as cases that can be timed and checked.

Every case is a dict of plain values.  "kind" names the call:

  iteration  one accelerated Lambda iteration as a driver loop writes it: the formal solve,
             then the statistical equilibrium (nlte_formal_solve_dev, nlte_stateq_dev)
  ali        a whole run from LTE to the tolerance (nlte_run_ali_dev), one or several models
  band       the same with the band ALO, which solves the coupled rate equations
  scatter    the formal solve with coherent scattering (nlte_formal_solve_scat_dev)
  trace      the walks of a new model's rays (nlte_trace), with what a driver reads of them
  rates      the statistical equilibrium alone over many points (nlte_stateq_dev)
  image      the emergent intensities of one line along one direction (nlte_image_dev)
  train      optimiser steps of the warm-start network (nlte_mlp_train_dev)
  predict    starting populations from the network (nlte_mlp_predict_dev)

"model" is one of the repository's three synthetic families: the static two-level sphere,
the five-level outflow and the ten-level Keplerian disc.  Inputs are made from the seed
alone, with their own generators here.  `exact` repeats each case's definition in FP64 with
torch and numpy (the walk, the second-order equation eliminated node by node, the rate
equations by LAPACK, the network without rounding).
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1912_08445_amd import binding

DEV = "cuda"
H, KB, C = 6.62607015e-27, 1.380649e-16, 2.99792458e10
AU, GM_SUN, AMU = 1.495978707e13, 1.32712440018e26, 1.66053906660e-24
T_CMB, F_SUB = 2.725, 0.25


# ------------------------------------------------------------------------------- cases

def listed():
    return [
        # The smallest problem of the repository: 1,000 points, 12 rays, one line.  Every
        # wave is a short chain and the launches count.
        dict(name="sphere_1k", kind="iteration", model="sphere", points=1000, nside=1, n_q=31, precision="fp64"),
        # The outflow at an ordinary size: long velocity sub-step segments.
        dict(name="outflow_20k", kind="iteration", model="outflow", points=20011, nside=2, n_q=31, precision="fp64"),
        # The disc, with the benchmark's 192 rays and 9 lines.
        dict(name="disc_30k", kind="iteration", model="disc", points=30011, nside=4, n_q=31, precision="fp64"),
        # The FP32-bulk option on the disc.
        dict(name="disc_24k_fp32", kind="iteration", model="disc", points=24007, nside=4, n_q=31, precision="fp32"),
        # A parameter study: ragged batch of outflows run to convergence in one call.
        dict(name="ali_batch", kind="ali", model="outflow", points=1500, models=9, nside=2, n_q=31,
             precision="fp64", tol=1e-4),
        # An optically thick sphere with the band operator: host-driven coupled solver.
        dict(name="band_3k", kind="band", model="sphere", points=3001, nside=1, n_q=31, tol=1e-6),
        # Scattering, on the uneven Gauss-Hermite offsets the paper uses.
        dict(name="scatter_5k", kind="scatter", model="outflow", points=5003, nside=2, n_q=24, quad="hermite"),
        # A new model's ray walks, paid once per model.
        dict(name="trace_50k", kind="trace", model="outflow", points=50000, nside=2),
        # The rate equations of a large ten-level model.
        dict(name="rates_200k", kind="rates", model="disc", points=200003),
        # A spectral cube of the disc.
        dict(name="image_40k", kind="image", model="disc", points=40009, nside=1, n_ch=64),
        # A stretch of the warm start's training at its own batch size.
        dict(name="train_4096", kind="train", rows=65536, batch=4096, steps=24, n_out=10),
        # The learned start of a new disc.
        dict(name="predict_40k", kind="predict", model="disc", points=40009, nside=2),
    ]


# Sizes (log-uniform) each kind is drawn from; the upper ends cost no more than the
# largest listed case.
RANGES = {
    ("iteration", "sphere"): (300, 60000), ("iteration", "outflow"): (500, 30000),
    ("iteration", "disc"): (1000, 30000), ("ali", "outflow"): (500, 2000), ("band", "sphere"): (300, 6000),
    ("scatter", "outflow"): (500, 6000), ("trace", "outflow"): (1000, 50000), ("trace", "disc"): (1000, 50000),
    ("rates", "outflow"): (5000, 300000), ("rates", "disc"): (5000, 250000),
    ("image", "outflow"): (2000, 40000), ("image", "disc"): (2000, 40000),
    ("predict", "outflow"): (2000, 40000), ("predict", "disc"): (2000, 40000),
}


def draw(rng):
    kind = rng.choice(["iteration", "iteration", "iteration", "iteration", "ali", "band", "scatter", "trace",
                       "rates", "image", "train", "predict"])
    if kind == "train":
        return dict(kind="train", rows=rng.randint(20000, 80000), batch=int(2 ** rng.uniform(7, 13)),
                    steps=rng.randint(8, 32), n_out=rng.choice([2, 5, 10, 16]))
    model = rng.choice([m for k, m in RANGES if k == kind])
    lo, hi = RANGES[kind, model]
    case = dict(kind=kind, model=model, points=int(round(lo * (hi / lo) ** rng.random())))
    if kind != "rates":
        case["nside"] = {"sphere": 1, "outflow": rng.choice([1, 2]), "disc": rng.choice([1, 2, 4])}[model]
        if kind in ("image", "trace", "predict"):
            case["nside"] = rng.choice([1, 2])
    if kind in ("iteration", "ali", "band", "scatter"):
        case["n_q"] = rng.choice([15, 24, 31, 31, 31, 47] if kind == "iteration" else [15, 24, 31])
    if kind in ("iteration", "ali"):
        case["precision"] = rng.choice(["fp64", "fp64", "fp32"])
    if kind == "scatter":
        case["quad"] = rng.choice(["uniform", "hermite"])
    if kind == "ali":
        case.update(models=rng.randint(1, 9), tol=1e-4)
    if kind == "band":
        case["tol"] = 1e-6
    if kind == "image":
        case["n_ch"] = rng.choice([21, 64, 100])
    return case


# ------------------------------------------------------------------------------ inputs

def _species(model):
    """Levels, lines and collision tables: the two-level species or a linear rotor."""
    T = np.geomspace(1.0, 5000.0, 48)
    law = 1e-10 * np.sqrt(T / 20.0)
    if model == "sphere":
        E, g = np.array([0.0, H * 100e9]), np.array([1.0, 3.0])
        up, lo, A = [1], [0], np.array([1e-5])
        pairs = [(1, 0)]
    else:
        n = 5 if model == "outflow" else 10
        J = np.arange(n, dtype=np.float64)
        E, g = H * 57.6e9 * J * (J + 1.0), 2.0 * J + 1.0
        up, lo = list(range(1, n)), list(range(n - 1))
        A = 7e-8 * 3.0 * J[1:] ** 4 / (2.0 * J[1:] + 1.0)
        pairs = [(u, l) for u in range(1, n) for l in range(u)]
    return SimpleNamespace(energy=E, weight=g, mass=28.0 * AMU, line_up=np.array(up, np.int32),
                           line_lo=np.array(lo, np.int32), line_A=A, coll_up=np.array([p[0] for p in pairs], np.int32),
                           coll_lo=np.array([p[1] for p in pairs], np.int32), coll_T=T,
                           coll_K=np.tile(law, (len(pairs), 1)), n_lev=len(E), n_lines=len(up))


def _knn(pos, k=12):
    """Exact k nearest neighbours, nearest first (distances from every point, on the GPU)."""
    p = torch.from_numpy(pos / np.abs(pos).max()).to(DEV)
    n, out = p.shape[0], []
    step = max(64, int(6e7) // n)
    for a in range(0, n, step):
        q = p[a:a + step]
        d = (q[:, None, 0] - p[None, :, 0]).square_()
        for c in (1, 2):
            d += (q[:, None, c] - p[None, :, c]).square_()
        d[torch.arange(q.shape[0], device=DEV), torch.arange(a, a + q.shape[0], device=DEV)] = math.inf
        out.append(d.topk(k, dim=1, largest=False).indices.to(torch.int32))
    return torch.cat(out).cpu().numpy()


def _model(family, n, rng, neighbours=True, scale_n=1.0, scale_T=1.0, thick=False):
    if family == "disc":
        R = 10.0 * AU * np.exp(rng.random(n) * math.log(50.0))
        phi = 2.0 * np.pi * rng.random(n)
        zeta = np.clip(rng.standard_normal(n), -3.0, 3.0)
        pos = np.stack([R * np.cos(phi), R * np.sin(phi), 0.1 * R * zeta], axis=1)
        n_h2 = 1.5e9 * (R / (10.0 * AU)) ** -2 * np.exp(-0.5 * zeta * zeta)
        T = 200.0 * (R / (10.0 * AU)) ** -0.5
        v = np.sqrt(GM_SUN / R)
        vel = np.stack([-v * np.sin(phi), v * np.cos(phi), np.zeros(n)], axis=1)
        X = 1e-6
    else:
        u = rng.standard_normal((n, 3))
        rhat = u / np.linalg.norm(u, axis=1)[:, None]
        r = 1e17 * rng.random(n) ** (1.0 / 3.0)
        pos = r[:, None] * rhat
        rr = np.maximum(r, 1e15) / 1e15
        if family == "sphere":
            n_h2, T, vel, X = 1e4 * rr ** -2.0, np.full(n, 20.0), np.zeros((n, 3)), 1e-6 if thick else 1e-8
        else:
            n_h2, T, vel, X = 1e7 * rr ** -2.0, 100.0 * rr ** -0.5, 15.0e5 * rhat, 1e-6
    if neighbours:
        nbr = _knn(pos)
    else:   # calls without rays: a ring
        i = np.arange(n, dtype=np.int32)
        nbr = np.stack([(i - 1) % n, (i + 1) % n], axis=1).astype(np.int32)
    return SimpleNamespace(pos=pos, vel=vel, n_h2=n_h2 * scale_n, temperature=T * scale_T, v_turb=np.full(n, 1.5e4),
                           abundance=np.full(n, X), nbr=nbr, boundary=None, n_points=n)


def _directions(nside):
    """HEALPix pixel centres, ring by ring; each with its antipode."""
    out = []
    for i in range(1, 4 * nside):
        if i < nside or i > 3 * nside:
            k = min(i, 4 * nside - i)
            z = (1.0 - k * k / (3.0 * nside * nside)) * (1 if i < nside else -1)
            phis = [(j - 0.5) * 0.5 * math.pi / k for j in range(1, 4 * k + 1)]
        else:
            z = (2 * nside - i) * 2.0 / (3.0 * nside)
            shift = 1.0 if (i + nside) % 2 else 0.5
            phis = [(j - shift) * math.pi / (2.0 * nside) for j in range(1, 4 * nside + 1)]
        s = math.sqrt(max(0.0, (1.0 - z) * (1.0 + z)))
        out += [(s * math.cos(p), s * math.sin(p), z) for p in phis]
    return np.array(out)


def _quadrature(n, kind="uniform"):
    if kind == "hermite":
        x, w = np.polynomial.hermite.hermgauss(n)
    else:
        x = np.linspace(-4.0, 4.0, n)
        w = np.exp(-x * x)
        w[0] *= 0.5
        w[-1] *= 0.5
    x, w = 0.5 * (x - x[::-1]), 0.5 * (w + w[::-1])
    return x, w / w.sum()


def _lte(sp, T, ntot):
    x = sp.weight * np.exp(-(sp.energy - sp.energy[0])[None, :] / (KB * T[:, None]))
    return ntot[:, None] * x / x.sum(axis=1, keepdims=True)


def _away_from_lte(sp, m, rng):
    """Populations in the middle of a run: upper levels under their LTE values, the more
    the higher and the thinner the gas, and a point's own scatter."""
    lte = _lte(sp, m.temperature, m.abundance * m.n_h2)
    thin = 1.0 / (1.0 + (m.n_h2 / 1e6) ** 0.5)[:, None]
    lev = np.arange(sp.n_lev)[None, :] / sp.n_lev
    p = lte * np.exp(-0.8 * thin * lev + 0.02 * rng.standard_normal(lte.shape))
    return p * (lte.sum(axis=1) / p.sum(axis=1))[:, None]


def _rng(case, seed):
    return np.random.default_rng([int(seed), int(case.get("points", case.get("rows", 0)))])


def _inputs(case, seed):
    rng = _rng(case, seed)
    i = SimpleNamespace(case=case, sp=_species(case["model"]), offsets=None)
    if case["kind"] == "ali":
        ms, off = [], [0]
        sizes = np.random.default_rng([case["points"], case["models"]])   # the study's, for every seed
        for _ in range(case["models"]):
            n = int(round(case["points"] * 3.0 ** sizes.uniform(-1.0, 1.0)))
            ms.append(_model("outflow", n, rng, scale_n=3.0 ** rng.uniform(-1, 1), scale_T=3.0 ** rng.uniform(-1, 1)))
            off.append(off[-1] + n)
        cat = {k: np.concatenate([getattr(m, k) for m in ms])
               for k in ("pos", "vel", "n_h2", "temperature", "v_turb", "abundance", "nbr")}
        i.m, i.offsets = SimpleNamespace(boundary=None, n_points=off[-1], **cat), np.array(off, np.int64)
    else:
        i.m = _model(case["model"], case["points"], rng, neighbours=case["kind"] != "rates",
                     thick=case["kind"] == "band")
    i.ntot = i.m.abundance * i.m.n_h2
    i.rays = _directions(case.get("nside", 1))
    i.x, i.w = _quadrature(case.get("n_q", 31), case.get("quad", "uniform"))
    if case["kind"] in ("iteration", "scatter", "rates", "image"):
        i.pops = _away_from_lte(i.sp, i.m, rng)
    if case["kind"] == "rates":
        # mean intensities between the background's and the gas's, and operators from
        # transparent to thick, as a formal solve of a disc leaves them
        B = _planck(_nu(i.sp)[None, :], i.m.temperature[:, None])
        dil = 10.0 ** rng.uniform(-3.0, 0.0, (i.m.n_points, 1))
        i.J = dil * B + (1.0 - dil) * _planck(_nu(i.sp), T_CMB)[None, :]
        i.L = rng.uniform(0.0, 0.95, i.J.shape)
        S = _line_coef(i)[1]
        i.Jeff = np.maximum(i.J - i.L * S, 0.05 * i.J)
    if case["kind"] == "scatter":
        kap = _line_coef(i)[0]
        i.chi_sca = np.broadcast_to(0.5 * np.median(kap, axis=0), kap.shape).copy()
        B0 = _planck(_nu(i.sp), T_CMB)[None, :, None]
        i.Jin = B0 * (1.0 + 5.0 * rng.random((i.m.n_points, i.sp.n_lines, 1)) * np.exp(-0.3 * i.x ** 2)[None, None, :])
    if case["kind"] == "image":
        n = i.rays[0]
        s = np.abs(i.m.vel @ n).max()
        i.v_ch = np.linspace(-1.0, 1.0, case["n_ch"]) * (s + 4.0 * _width(i).max())
    if case["kind"] == "predict":
        i.theta = _weights(rng, i.sp.n_lev)
        i.mean = np.array([6.0, 1.8, -9.0, 20.0, 21.0, 21.5, 22.0, 22.5])
        i.std = np.array([1.5, 0.3, 0.7, 1.5, 1.2, 1.0, 1.0, 1.0])
    return i


def _nu(sp):
    return (sp.energy[sp.line_up] - sp.energy[sp.line_lo]) / H


def _planck(nu, T):
    return 2.0 * H * nu ** 3 / C ** 2 / np.expm1(H * nu / (KB * T))


def _width(i):
    return np.sqrt(2.0 * KB * i.m.temperature / i.sp.mass + i.m.v_turb ** 2)


def _einstein(sp):
    nu = _nu(sp)
    Bul = sp.line_A * C ** 2 / (2.0 * H * nu ** 3)
    return nu, Bul, Bul * sp.weight[sp.line_up] / sp.weight[sp.line_lo]


def _line_coef(i, pops=None):
    """Line-centre opacity and source function per point and line."""
    p = i.pops if pops is None else pops
    nu, Bul, Blu = _einstein(i.sp)
    nup, nlo = p[:, i.sp.line_up], p[:, i.sp.line_lo]
    chi = H * nu / (4.0 * math.pi) * (nlo * Blu - nup * Bul)
    eta = H * nu / (4.0 * math.pi) * nup * i.sp.line_A
    on = chi > 0.0
    kap = np.where(on, chi / (math.sqrt(math.pi) * nu * _width(i)[:, None] / C), 0.0)
    return kap, np.where(on, eta / np.where(on, chi, 1.0), 0.0)


def _weights(rng, n_out):
    parts = []
    for a, b in ((8, 128), (128, 128), (128, 128), (128, n_out)):
        parts += [rng.uniform(-1, 1, a * b) * math.sqrt(6.0 / (a + b)) * (0.3 if b == n_out else 1.0),
                  0.02 * rng.standard_normal(b)]
    return np.concatenate(parts).astype(np.float32)


def _rows(case, seed):
    """Standardised features and smooth departures from LTE with a little scatter."""
    rng = _rng(case, seed)
    X = rng.standard_normal((case["rows"], 8)).astype(np.float32)
    W = rng.standard_normal((8, case["n_out"])) / math.sqrt(8.0)
    T = (0.5 * np.tanh(X @ W) + 0.01 * rng.standard_normal((case["rows"], case["n_out"]))).astype(np.float32)
    return X, T, _weights(rng, case["n_out"])


# ---------------------------------------------------------------------- prepare and run

def _solver(i):
    case, s = i.case, binding.Solver(0)
    s.set_species(i.sp)
    s.set_models(i.m, i.offsets)
    s.set_rays(i.rays)
    s.set_quadrature(i.x, i.w)
    s.set_params(t_cmb=T_CMB, f_sub=F_SUB, max_iter=60, tol=case.get("tol", 1e-4),
                 precision=case.get("precision", "fp64"), alo_band=int(case["kind"] == "band"))
    return s


def prepare(case, seed):
    st = SimpleNamespace(kind=case["kind"])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    if case["kind"] == "train":
        X, T, theta = _rows(case, seed)
        st.s = binding.Solver(0)
        st.s.mlp_set_weights(theta, case["n_out"])
        st.X, st.T, st.steps, st.batch = dev(X), dev(T), case["steps"], case["batch"]
        st.curve = torch.empty(case["steps"], dtype=torch.float32, device=DEV)
        return st
    i = _inputs(case, seed)
    st.s = s = _solver(i)
    if case["kind"] not in ("trace", "rates"):
        s.trace()
    P, nl, n = i.m.n_points, i.sp.n_lines, i.sp.n_lev
    new = lambda *shape: torch.empty(shape, dtype=torch.float64, device=DEV)  # noqa: E731
    st.out = new(P, n)
    if case["kind"] in ("iteration", "scatter", "rates", "image"):
        st.pops = dev(i.pops)
    if case["kind"] in ("iteration", "scatter"):
        st.J, st.Jeff, st.L = new(P, nl), new(P, nl), new(P, nl)
    if case["kind"] in ("iteration", "rates"):
        st.flags = torch.empty(P, dtype=torch.uint8, device=DEV)
    if case["kind"] == "rates":
        st.J, st.Jeff, st.L = dev(i.J), dev(i.Jeff), dev(i.L)
    if case["kind"] == "scatter":
        s.set_scattering(i.chi_sca)
        st.Jin, st.Jout = dev(i.Jin), new(P, nl, len(i.x))
    if case["kind"] == "image":
        st.v, st.I, st.xy, st.line = i.v_ch, new(P, case["n_ch"]), new(P, 2), min(2, nl - 1)
    if case["kind"] == "predict":
        s.mlp_set_weights(i.theta, n)
        s.mlp_set_norm(i.mean, i.std)
    return st


def run(st):
    s, kind = st.s, st.kind
    if kind == "iteration":
        s.formal_solve_dev(st.pops, st.J, st.Jeff, st.L)
        s.stateq_dev(st.pops, st.J, st.Jeff, st.L, st.out, st.flags)
        return [st.J, st.Jeff, st.L, st.out, st.flags]
    if kind in ("ali", "band"):
        rep = s.run_ali_dev(None, st.out)
        return [st.out, rep["iterations"]]
    if kind == "scatter":
        s.formal_solve_scat_dev(st.pops, st.Jin, st.J, st.Jeff, st.L, st.Jout)
        return [st.J, st.Jeff, st.L, st.Jout]
    if kind == "trace":
        s.trace()
        return [s.point_cost(), *s.trace_stats()]
    if kind == "rates":
        s.stateq_dev(st.pops, st.J, st.Jeff, st.L, st.out, st.flags)
        return [st.out, st.flags]
    if kind == "image":
        s.image_dev(st.pops, 0, st.line, st.v, st.I, st.xy)
        return [st.I, st.xy]
    if kind == "train":
        s.mlp_train_dev(st.X, st.T, st.curve, steps=st.steps, batch=st.batch, lr=2e-4)
        return [st.curve, s.mlp_get_weights()]
    return [st.out, s.mlp_predict_dev(st.out)]


def work(case):
    """Bytes and operations that no implementation can leave out.  The lengths of the
    walks are those of the families (cells per ray 0.95 P^(1/3) in a ball, 0.9 P^(1/3) in
    the disc); an elimination step of one line at one frequency is 17 FP64 operations."""
    if case["kind"] == "train":
        rows, n = case["batch"] * case["steps"], case["n_out"]
        weights = 8 * 128 + 2 * 128 * 128 + 128 * n
        return {"bytes": rows * (8 + n) * 4 + case["steps"] * weights * 24.0, "flops": 6.0 * rows * weights}
    sp, P = _species(case["model"]), case["points"] * case.get("models", 1)
    nl, n = sp.n_lines, sp.n_lev
    rays = 12 * case.get("nside", 1) ** 2
    cells = (0.9 if case["model"] == "disc" else 0.95) * case["points"] ** (1.0 / 3.0)
    # elimination steps per ray: its cells, plus the velocity sub-steps that any lane needs
    steps = {"sphere": cells, "outflow": cells + 150.0, "disc": 1.3 * cells}[case["model"]]
    rate_flops = 2.0 / 3.0 * n ** 3 + 40.0 * len(sp.coll_up)
    fields = P * (64.0 + 16.0 * nl)
    if case["kind"] == "rates":
        return {"bytes": P * (16.0 * n + 24.0 * nl + 24.0), "flops": P * rate_flops}
    if case["kind"] == "trace":
        return {"bytes": P * (64.0 + 48.0) + P * rays * (8.0 + 4.0 * cells), "flops": P * rays * cells * 12 * 20.0}
    if case["kind"] == "predict":
        return {"bytes": fields + P * rays * (8.0 + 4.0 * cells) + 8.0 * P * n,
                "flops": P * (rays * cells * 12.0 + 2.0 * (8 * 128 + 2 * 128 * 128 + 128 * n))}
    if case["kind"] == "image":
        return {"bytes": fields + 8.0 * P * (case["n_ch"] + 2) + 8.0 * P * cells,
                "flops": 17.0 * P * 2.0 * steps * case["n_ch"]}
    sweep = {"bytes": fields + P * rays * (8.0 + 4.0 * cells) + 8.0 * P * (3 * nl + 2 * n),
             "flops": 17.0 * P * rays * steps * nl * case["n_q"] + P * rate_flops}
    if case["kind"] == "scatter":
        return {"bytes": sweep["bytes"] + 16.0 * P * nl * case["n_q"], "flops": 2.0 * sweep["flops"]}
    times = {"ali": 3, "band": 8}.get(case["kind"], 1)
    return {"bytes": times * sweep["bytes"], "flops": times * sweep["flops"]}


# ------------------------------------------------------------------------------- exact

def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] in ("trace", "band"):
        return None   # whole numbers; a coupled solve whose iterates depend on its operator
    i = _inputs(case, seed)
    if case["kind"] == "rates":
        return [_stateq(i, i.Jeff, i.L), None]
    g = _Walks(i)
    if case["kind"] == "iteration":
        J, Jeff, L = g.solve(i.pops)
        return [J, Jeff, L, _stateq(i, Jeff, L), None]
    if case["kind"] == "ali":
        return _exact_ali(i, g)
    if case["kind"] == "scatter":
        return g.solve(i.pops, scatter=True)
    if case["kind"] == "image":
        return g.image(i)
    return _exact_predict(i, g)


def _stateq(i, Jeff, L):
    """Populations of the rate equations with the diagonal operator, one LAPACK solve each."""
    sp, m, P, n = i.sp, i.m, i.m.n_points, i.sp.n_lev
    nu, Bul, Blu = _einstein(sp)
    M = np.zeros((P, n, n))

    def rate(a, b, R):   # a -> b
        M[:, b, a] += R
        M[:, a, a] -= R

    for l, (u, lo) in enumerate(zip(sp.line_up, sp.line_lo)):
        rate(u, lo, sp.line_A[l] * (1.0 - L[:, l]) + Bul[l] * Jeff[:, l])
        rate(lo, u, Blu[l] * Jeff[:, l])
    for c, (u, lo) in enumerate(zip(sp.coll_up, sp.coll_lo)):
        K = np.interp(m.temperature, sp.coll_T, sp.coll_K[c]) * m.n_h2
        rate(u, lo, K)
        rate(lo, u, K * sp.weight[u] / sp.weight[lo] * np.exp(-(sp.energy[u] - sp.energy[lo]) / (KB * m.temperature)))
    M[:, 0, :] = 1.0
    b = np.zeros((P, n, 1))
    b[:, 0, 0] = i.ntot
    return np.linalg.solve(M, b)[:, :, 0]


def _exact_ali(i, g):
    p = _lte(i.sp, i.m.temperature, i.ntot)
    done = np.zeros(len(i.offsets) - 1, bool)
    it = 0
    while it < 60 and not done.all():
        J, Jeff, L = g.solve(p)
        q = _stateq(i, Jeff, L)
        it += 1
        change = np.where(q / i.ntot[:, None] > 1e-10, np.abs(q - p) / q, 0.0).max(axis=1)
        for k in range(len(done)):
            sl = slice(i.offsets[k], i.offsets[k + 1])
            if not done[k]:
                p[sl] = q[sl]
                done[k] = change[sl].max() < i.case["tol"]
    return [p, it]


class _Walks:
    """All walks of a model and the eliminations along them, in FP64 on the GPU."""

    def __init__(self, i):
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
        self.i = i
        self.pos, self.vel, self.vw = t(i.m.pos), t(i.m.vel), t(_width(i))
        self.x, self.w = t(i.x), t(i.w)
        self.dirs = t(i.rays)
        self.P, self.R = i.m.n_points, i.rays.shape[0]
        off = np.zeros(self.P, np.int64) if i.offsets is None else np.repeat(i.offsets[:-1], np.diff(i.offsets))
        nbr = t(i.m.nbr.astype(np.int64) + off[:, None])
        n = self.P * self.R
        O = torch.arange(n, device=DEV) // self.R
        d = self.dirs.repeat(self.P, 1)
        self.len = torch.zeros(n, dtype=torch.int64, device=DEV)
        cur, z, act, cells = O.clone(), torch.zeros(n, dtype=torch.float64, device=DEV), torch.arange(n, device=DEV), []
        while act.numel():
            col = torch.full((n,), -1, dtype=torch.int32, device=DEV)
            keep = []
            for a in act.split(1 << 20):
                m = nbr[cur[a]]
                r, u = self.pos[m] - self.pos[O[a]][:, None, :], d[a][:, None, :]
                Z = (r[..., 0] * u[..., 0] + r[..., 1] * u[..., 1]) + r[..., 2] * u[..., 2]
                e = r - Z[..., None] * u
                q = (e[..., 0] * e[..., 0] + e[..., 1] * e[..., 1]) + e[..., 2] * e[..., 2]
                q = torch.where(Z > z[a][:, None], q, math.inf)
                best, s = q.min(dim=1)
                ok = torch.isfinite(best)
                a, s = a[ok], s[ok]
                cur[a] = m[ok].gather(1, s[:, None])[:, 0]
                z[a] = Z[ok].gather(1, s[:, None])[:, 0]
                col[a] = cur[a].to(torch.int32)
                self.len[a] += 1
                keep.append(a)
            act = torch.cat(keep)
            if act.numel():
                cells.append(col)
        self.cells = torch.stack(cells, dim=1) if cells else torch.zeros((n, 0), dtype=torch.int32, device=DEV)

    def _half(self, rays):
        """Base nodes of half rays from the far end to the origin (left aligned, the origin
        repeated beyond it): cell, projection, projected velocity."""
        L = int(self.len[rays].max()) if rays.numel() else 0
        O = rays // self.R
        k = self.len[rays][:, None] - 1 - torch.arange(L + 1, device=DEV)[None, :]
        c = self.cells[rays].to(torch.int64).gather(1, k.clamp(min=0)) if L else k.clone()
        c = torch.where(k >= 0, c, O[:, None])
        u = self.dirs[rays % self.R][:, None, :]
        r, v = self.pos[c] - self.pos[O][:, None, :], self.vel[c] - self.vel[O][:, None, :]
        return c, (r * u).sum(-1), (v * u).sum(-1)

    def _parts(self, c, s, n_base):
        """Sub-intervals of every base segment (0 past the last)."""
        w = self.vw[c]
        ds, thr = (s[:, 1:] - s[:, :-1]).abs(), F_SUB * torch.minimum(w[:, 1:], w[:, :-1])
        m = torch.where(ds > thr, torch.ceil(ds / thr), torch.ones_like(ds)).to(torch.int64)
        return torch.where(torch.arange(m.shape[1], device=DEV)[None, :] < n_base[:, None], m, torch.zeros_like(m))

    def _fine(self, m, t):
        """(segment, fraction) of fine node t of every ray; the last node at the end."""
        cum = m.cumsum(1)
        seg = torch.searchsorted(cum, torch.full_like(cum[:, :1], t), right=True)[:, 0].clamp(max=m.shape[1] - 1)
        mm = m.gather(1, seg[:, None])[:, 0].clamp(min=1)
        j = t - (cum.gather(1, seg[:, None])[:, 0] - m.gather(1, seg[:, None])[:, 0])
        return seg, (j.to(torch.float64) / mm).clamp(max=1.0)

    def _sorted_chunks(self, total, width):
        order = torch.argsort(total)
        step = max(256, int(1.5e7) // width)
        return order.split(step)

    def solve(self, pops, scatter=False):
        i, nl, nq = self.i, self.i.sp.n_lines, len(self.i.x)
        kap, S = (torch.from_numpy(a).to(DEV) for a in _line_coef(i, pops))
        I0 = torch.from_numpy(_planck(_nu(i.sp), T_CMB)).to(DEV)[None, :, None]
        n = self.P * self.R
        chi_s = torch.from_numpy(i.chi_sca).to(DEV) if scatter else None
        Jin = torch.from_numpy(i.Jin).to(DEV) if scatter else None
        up = self._upper()
        keys = ("Q", "y", "D") + (("yv", "sg", "Sp") if scatter else ())
        res = {k: torch.empty((n, nl, nq), dtype=torch.float64, device=DEV) for k in keys}
        total = torch.empty(n, dtype=torch.int64, device=DEV)
        for rays in torch.arange(n, device=DEV).split(1 << 18):
            c, _, s = self._half(rays)
            total[rays] = self._parts(c, s, self.len[rays]).sum(1)
        for rays in self._sorted_chunks(total, nl * nq):
            c, z, s = self._half(rays)
            if c.shape[1] == 1:     # no cell on any of these rays
                c, z, s = (v.repeat(1, 2) for v in (c, z, s))
            m = self._parts(c, s, self.len[rays])
            N = int(total[rays].max())
            sign = torch.where(up[rays % self.R], -1.0, 1.0).to(torch.float64)
            a = self.vw[rays // self.R][:, None] / self.vw[c]
            b = s / self.vw[c]
            xq = sign[:, None] * self.x[None, :]
            sh = (len(rays), nl, nq)
            Q, y, D = torch.ones(sh, dtype=torch.float64, device=DEV), I0.expand(sh).clone(), torch.zeros(sh, dtype=torch.float64, device=DEV)
            yv = -sign[:, None, None] * I0.expand(sh)   # the background enters with -v at the ahead end
            prev = None
            for t in range(N + 1):
                seg, f = self._fine(m, t)
                at = lambda v: v.gather(1, seg[:, None])[:, 0], lambda v: v.gather(1, (seg + 1).clamp(max=v.shape[1] - 1)[:, None])[:, 0]  # noqa: E731
                lin = lambda v: at[0](v) + f * (at[1](v) - at[0](v))  # noqa: E731
                c0, c1, ff = at[0](c), at[1](c), f[:, None]
                zt = lin(z)
                yx = lin(a)[:, None] * xq - lin(b)[:, None]
                k = kap[c0] + ff * (kap[c1] - kap[c0])
                St = (S[c0] + ff * (S[c1] - S[c0]))[:, :, None].expand(sh)
                chi = k[:, :, None] * torch.exp(-yx * yx)[:, None, :]
                sg = None
                if scatter:
                    yz = sign[:, None] * yx      # in the pair's own orientation
                    cs = (chi_s[c0] + ff * (chi_s[c1] - chi_s[c0]))[:, :, None]
                    jp = (1 - ff[..., None]) * self._at(Jin, c0, yz) + ff[..., None] * self._at(Jin, c1, yz)
                    jm = (1 - ff[..., None]) * self._at(Jin, c0, -yz) + ff[..., None] * self._at(Jin, c1, -yz)
                    tot = chi + cs
                    on = tot > 0
                    den = torch.where(on, tot, 1.0)
                    St = torch.where(on, (chi / den) * St + cs / den * 0.5 * (jp + jm), St)
                    sg = torch.where(on, cs / den * 0.5 * (jp - jm), 0.0)
                    chi = tot
                if prev is not None:
                    # eliminate the previous node, whose neighbours are pp (before) and this
                    live = (t <= total[rays])[:, None, None]
                    z0, chi0, S0, sg0 = prev[:4]
                    Dn = 0.5 * (chi0 + chi) * (z0 - zt)[:, None, None]
                    h = 0.5 * (D + Dn)
                    E = 1.0 / (1.0 + Dn * (h + Q))
                    r = h * S0 + y
                    if scatter:
                        e = -0.5 * sign[:, None, None]   # rows take differences along the pair's direction
                        r = r - e * (sg - prev[5])
                        rv = h * sg0 + yv - e * (St - prev[4])
                        yv = torch.where(live, rv * E, yv)
                    y, Q = torch.where(live, r * E, y), torch.where(live, (h + Q) * E, Q)
                    D = torch.where(live, Dn, D)
                    if scatter:    # sources of the last node before the origin
                        Sl, sl = torch.where(live, S0, prev[6]), torch.where(live, sg0, prev[7])
                        prev = (zt, chi, St, sg, S0, sg0, Sl, sl)
                    else:
                        prev = (zt, chi, St, None)
                else:
                    prev = (zt, chi, St, sg) + ((-St, -sg, -St, -sg) if scatter else ())
            res["Q"][rays], res["y"][rays], res["D"][rays] = Q, y, D
            if scatter:
                res["yv"][rays], res["Sp"][rays], res["sg"][rays] = yv, prev[6], prev[7]
        return self._combine(res, kap, S, chi_s, Jin, scatter)

    def _upper(self):
        """Rays behind the origin along their pair's direction (the antipode, whose index is lower, points ahead)."""
        anti = torch.cdist(self.dirs, -self.dirs).argmin(1)
        self.anti = anti
        return anti < torch.arange(self.R, device=DEV)

    def _at(self, Jin, c, y):
        """The field of cells c at offsets y: linear between the quadrature's, constant beyond."""
        x, nq = self.x, len(self.x)
        j = (torch.searchsorted(x, y.contiguous(), right=True) - 1).clamp(0, nq - 2)
        f = ((y - x[j]) / (x[j + 1] - x[j])).clamp(0.0, 1.0)[:, None, :]
        row = Jin[c]
        j = j[:, None, :].expand(-1, row.shape[1], -1)
        lo = row.gather(2, j)
        return lo + f * (row.gather(2, j + 1) - lo)

    def _combine(self, res, kap, S, chi_s, Jin, scatter):
        """Both halves of every pair at the origin, and the sums over pairs and frequencies."""
        P, R, nl, nq = self.P, self.R, S.shape[1], len(self.x)
        J, Jeff, L = (torch.zeros((P, nl), dtype=torch.float64, device=DEV) for _ in range(3))
        Jp, Jm = (torch.zeros((P, nl, nq), dtype=torch.float64, device=DEV) for _ in range(2))
        v = {k: a.view(P, R, nl, nq) for k, a in res.items()}
        So, line = S[:, :, None], kap[:, :, None] * torch.exp(-self.x * self.x)[None, None, :]
        share, sgo, Spo = torch.ones_like(line), None, So.expand_as(line)
        if scatter:
            cs = chi_s[:, :, None]
            tot = line + cs
            on = tot > 0
            den = torch.where(on, tot, 1.0)
            share = torch.where(on, line / den, 1.0)
            jm = Jin.flip(2)
            Spo = torch.where(on, share * So + cs / den * 0.5 * (Jin + jm), So)
            sgo = torch.where(on, cs / den * 0.5 * (Jin - jm), 0.0)
        for r in range(R):
            b = int(self.anti[r])
            if b < r:
                continue
            # the frequencies of the half behind run in the pair's orientation already
            h = 0.5 * (v["D"][:, r] + v["D"][:, b])
            inv = 1.0 / (h + v["Q"][:, r] + v["Q"][:, b])
            y = v["y"][:, r] + v["y"][:, b]
            rest = y
            if scatter:
                rest = y - self._slope(v["sg"], r, b, sgo)
                uo = (h * Spo + rest) * inv
                vo = (h * sgo + v["yv"][:, r] + v["yv"][:, b] - self._slope(v["Sp"], r, b, Spo)) * inv
                Jp += uo + vo
                Jm += uo - vo
            else:
                uo = (h * Spo + rest) * inv
            lam = h * inv * share
            J += (uo * self.w).sum(2)
            L += (lam * self.w).sum(2)
            Jeff += ((y * inv if not scatter else uo - lam * So) * self.w).sum(2)
        out = [a.mul(2.0 / R).cpu().numpy() for a in (J, Jeff, L)]
        return out + [((Jp + Jm.flip(2)) / R).cpu().numpy()] if scatter else out

    def _slope(self, last, r, b, own):
        """Half the difference of a quantity across the origin: the half behind lies before it
        along the pair's direction; an empty half mirrors the origin's value."""
        O = torch.arange(self.P, device=DEV) * self.R
        ahead = torch.where((self.len[O + r] > 0)[:, None, None], last[:, r], -own)
        behind = torch.where((self.len[O + b] > 0)[:, None, None], last[:, b], -own)
        # the ray r of a pair points to larger z: its nodes are eliminated toward smaller z
        return 0.5 * (ahead - behind)

    def image(self, i):
        line = min(2, i.sp.n_lines - 1)
        kap, S = (torch.from_numpy(a[:, line].copy()).to(DEV) for a in _line_coef(i))
        I_in = float(_planck(_nu(i.sp)[line], T_CMB))
        n = self.dirs[0]
        self._upper()
        f, b = torch.arange(self.P, device=DEV) * self.R, torch.arange(self.P, device=DEV) * self.R + self.anti[0]
        v = torch.from_numpy(i.v_ch).to(DEV)
        out = torch.empty((self.P, len(v)), dtype=torch.float64, device=DEV)
        nb, nf = self.len[b], self.len[f]
        k = torch.arange(int((nb + nf).max()) + 1, device=DEV)[None, :]
        back = self.cells[b].to(torch.int64).gather(1, (nb[:, None] - 1 - k).clamp(0, self.cells.shape[1] - 1))
        ahead = self.cells[f].to(torch.int64).gather(1, (k - nb[:, None] - 1).clamp(0, self.cells.shape[1] - 1))
        O = torch.arange(self.P, device=DEV)[:, None]
        c = torch.where(k < nb[:, None], back, torch.where(k == nb[:, None], O, ahead))
        last = c.gather(1, (nb + nf)[:, None])
        c = torch.where(k <= (nb + nf)[:, None], c, last)
        z, s = ((self.pos[c] - self.pos[O]) * n).sum(-1), ((self.vel[c] - self.vel[O]) * n).sum(-1)
        m = self._parts(c, s, nb + nf)
        total = m.sum(1)
        for p in self._sorted_chunks(total, len(v)):
            mm, N = m[p], int(total[p].max())
            a, bb = self.vw[p][:, None] / self.vw[c[p]], s[p] / self.vw[c[p]]
            xO = (v[None, :] - (self.vel[p] * n).sum(-1)[:, None]) / self.vw[p][:, None]
            Q = torch.ones((len(p), len(v)), dtype=torch.float64, device=DEV)
            y, D, prev = Q * I_in, Q * 0.0, None
            for t in range(N + 1):
                seg, fr = self._fine(mm, t)
                lin = lambda q: (lambda q0, q1: q0 + fr * (q1 - q0))(q.gather(1, seg[:, None])[:, 0], q.gather(1, seg[:, None] + 1)[:, 0])  # noqa: E731
                x = lin(a)[:, None] * xO - lin(bb)[:, None]
                chi, St, zt = lin(kap[c[p]])[:, None] * torch.exp(-x * x), lin(S[c[p]])[:, None], lin(z[p])
                if prev is not None:
                    live = (t <= total[p])[:, None]
                    Dn = 0.5 * (prev[1] + chi) * (zt - prev[0])[:, None]
                    h = 0.5 * (D + Dn)
                    E = 1.0 / (1.0 + Dn * (h + Q))
                    y, Q = torch.where(live, (h * prev[2] + y) * E, y), torch.where(live, (h + Q) * E, Q)
                    D = torch.where(live, Dn, D)
                prev = (zt, chi, St)
            u = (0.5 * D * prev[2] + y + I_in) / (0.5 * D + Q + 1.0)
            out[p] = 2.0 * u - I_in
        d = i.rays[0]
        ref = np.array([1.0, 0.0, 0.0]) if abs(d[2]) > 0.9 else np.array([0.0, 0.0, 1.0])
        e1 = np.cross(ref, d)
        e1 /= np.linalg.norm(e1)
        return [out.cpu().numpy(), np.stack([i.m.pos @ e1, i.m.pos @ np.cross(d, e1)], axis=1)]

    def features(self, i):
        nh2 = torch.from_numpy(i.m.n_h2).to(DEV)
        col = torch.empty(self.P * self.R, dtype=torch.float64, device=DEV)
        for rays in torch.arange(self.P * self.R, device=DEV).split(1 << 18):
            c, z, _ = self._half(rays)
            d = nh2[c]
            col[rays] = (0.5 * (d[:, 1:] + d[:, :-1]) * (z[:, :-1] - z[:, 1:])).sum(1)
        nbr = torch.from_numpy(i.m.nbr.astype(np.int64)).to(DEV)
        dx = (self.pos[nbr] - self.pos[:, None]).norm(dim=2)
        dv = (self.vel[nbr] - self.vel[:, None]).norm(dim=2)
        floor = (0.5 * nh2 * dx.mean(1)).clamp(min=1.0)
        col = torch.maximum(col.view(self.P, self.R), floor[:, None])
        q = torch.quantile(col, torch.tensor([0.0, 0.25, 0.5, 0.75, 1.0], dtype=torch.float64, device=DEV), dim=1).T
        T = torch.from_numpy(i.m.temperature).to(DEV)
        return torch.cat([nh2.log10()[:, None], T.log10()[:, None],
                          (dv / dx).mean(1).clamp(min=1e-30).log10()[:, None], q.log10()], dim=1)


def _layers(theta, n_out):
    out, o = [], 0
    for a, b in ((8, 128), (128, 128), (128, 128), (128, n_out)):
        out += [theta[o:o + a * b].view(b, a), theta[o + a * b:o + a * b + b]]
        o += a * b + b
    return out


def _net(theta, n_out, X):
    w = _layers(theta, n_out)
    h = X
    for k in range(4):
        h = h @ w[2 * k].T + w[2 * k + 1]
        if k < 3:
            h = torch.nn.functional.gelu(h)
    return h


def _exact_predict(i, g):
    F = (g.features(i) - torch.from_numpy(i.mean).to(DEV)) / torch.from_numpy(i.std).to(DEV)
    y = _net(torch.from_numpy(i.theta).to(DEV).double(), i.sp.n_lev, F).cpu().numpy()
    p = _lte(i.sp, i.m.temperature, i.ntot) * 10.0 ** y
    return [p * (i.ntot / p.sum(axis=1))[:, None], 0]


def _exact_train(case, seed):
    """The same steps of Adam on the network without rounding."""
    X, T, theta = (torch.from_numpy(a).to(DEV).double() for a in _rows(case, seed))
    theta.requires_grad_(True)
    opt, curve = torch.optim.Adam([theta], lr=2e-4, betas=(0.9, 0.999), eps=1e-8), []
    for k in range(case["steps"]):
        rows = (k * case["batch"] + torch.arange(case["batch"], device=DEV)) % case["rows"]
        opt.zero_grad()
        loss = (_net(theta, case["n_out"], X[rows]) - T[rows]).square().mean()
        loss.backward()
        opt.step()
        curve.append(float(loss.detach()))
    return [np.array(curve), theta.detach().cpu().numpy()]
