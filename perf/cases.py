"""Timing cases of the VEGAS framework: what a program that uses it has it do, through
its public entry points (Integrator, vegas_sigma, Flow), over the range of sizes that
such programs have.

Kinds of cases:
  integrate   a whole calculation on a new handle, from the uniform grid: iterations,
              refinements, the combined result, the final grid (a point of a parameter
              scan; small ones are bound by launches, host calls and latency)
  proceed     production iterations of a kept handle from a checkpoint of an adapted
              grid (the usual, long part of a calculation)
  schedule    the same through run_schedule: the two-stage schedule of the paper's runs
  grad        sigma and its gradient for a batch of Drell-Yan parameter points (a fit
              to data), forward and backward through autograd
  train       Adam steps of the learned proposal on weighted events
  loss_grad   its loss and gradient alone (a caller with an optimiser of its own)
  density     log q of given points (validation of a trained proposal)
  sample      proposal points from uniform ones
  flow_iterate  one iteration with the learned proposal in place of the grid's points

The inputs are the repository's named workloads (workloads.py) under a seed; exact()
restates the method in plain binary64 PyTorch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1503_06182_amd as P
import workloads as W
from paper_1503_06182_amd import flow as F

GRID_ADAPT = (4, 100_000)     # iterations and events that adapt the grid of a kept handle
BATCH_MAX = 1 << 18           # largest batch a density / gradient case asks for
FLOPS_EVENT = {"dy_z": 300.0, "w_plus": 373.5, "ww_4l": 1262.7, "ww_had": 1589.8}
FLOPS_GRAD_POINT = 100.0      # one parameter point of one event: a propagator, a power, six sums
FLOPS_FLOW_EVENT = 6 * 2.0 * (4 * 128 + 128 * 128 + 128 * 188)


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a point of a parameter scan: a new handle, the configuration's five iterations,
        # each read back by the program; latency and launches count
        dict(name="dy_z_scan_point", kind="integrate", workload="dy_z", n=10_000, iters=5, read=True,
             obs=0, strata=0, beta=0.0, fp32=False),
        # the two-stage schedule of the paper's timing runs, 4 x 1,000 + 10 x 10,000 events
        dict(name="ww_4l_paper_schedule", kind="schedule", workload="ww_4l", n1=1000, k1=4, n2=10_000, k2=10),
        # pp -> W+ with cuts at its configured size, with the lepton pT distribution
        dict(name="w_plus_observable", kind="integrate", workload="w_plus", n=1_000_000, iters=10, read=False,
             obs=50, strata=0, beta=0.0, fp32=False),
        # the flagship integrand at its configured size, on an adapted grid
        dict(name="ww_4l_production", kind="proceed", workload="ww_4l", n=10_000_000, iters=5, read=False,
             strata=0, beta=0.0, fp32=False),
        # the hadronic 10-dimensional integrand, a ragged event count
        dict(name="ww_had_production", kind="proceed", workload="ww_had", n=3_000_017, iters=3, read=True,
             strata=0, beta=0.0, fp32=False),
        # stratified + importance sampling with equal counts per hypercube
        dict(name="w_plus_strata", kind="proceed", workload="w_plus", n=1_000_000, iters=5, read=False,
             strata=26, beta=0.0, fp32=False),
        # adaptive allocation over the hypercubes
        dict(name="ww_4l_strata_adaptive", kind="proceed", workload="ww_4l", n=1_000_003, iters=4, read=False,
             strata=4, beta=0.75, fp32=False),
        # a fit's gradient: 64 parameter points at the published example's event count
        dict(name="grad_64_points", kind="grad", points=64, n=1_000_000),
        # a few points on a smaller, ragged sample
        dict(name="grad_9_points", kind="grad", points=9, n=100_003),
        # training of the learned proposal, the default batch
        dict(name="flow_train", kind="train", n=200_003, batch=4096, steps=10),
        # log q of a validation sample, a ragged batch
        dict(name="flow_density", kind="density", n=200_003),
        # a production iteration with the learned proposal
        dict(name="flow_iterate", kind="flow_iterate", n=1_000_003),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["integrate", "integrate", "proceed", "proceed", "proceed", "schedule", "grad", "grad",
                       "train", "loss_grad", "density", "sample", "flow_iterate"])
    if kind in ("integrate", "proceed"):
        workload = rng.choice(["dy_z", "w_plus", "ww_4l", "ww_had"])
        c = dict(kind=kind, workload=workload, n=_log_int(rng, 1000, 3_000_000), iters=rng.randint(1, 8),
                 read=rng.random() < 0.5, strata=0, beta=0.0, fp32=workload == "ww_4l" and rng.random() < 0.25)
        if kind == "integrate":
            c["obs"] = rng.choice([0, 0, 20, 50, 101])
        else:
            c["iters"] = min(c["iters"], 5)
            if rng.random() < 0.4:
                c["beta"] = rng.choice([0.0, 0.75])
                per = 8 if c["beta"] else rng.choice([2, 5])
                m = int((c["n"] / per) ** (1.0 / W.NDIM[W.config(workload)["process"]]) + 1e-9)
                c["strata"] = max(1, m)
        if kind == "integrate":
            c["strata"], c["beta"] = 0, 0.0
        return c
    if kind == "schedule":
        return dict(kind=kind, workload=rng.choice(["dy_z", "w_plus", "ww_4l"]), n1=_log_int(rng, 500, 5000),
                    k1=2 * rng.randint(1, 3), n2=_log_int(rng, 5000, 100_000), k2=2 * rng.randint(1, 5))
    if kind == "grad":
        return dict(kind=kind, points=rng.choice([1, 2, 7, 16, 33, 64]), n=_log_int(rng, 2000, 1_000_000))
    if kind == "train":
        return dict(kind=kind, n=_log_int(rng, 20_000, 1_000_000), batch=_log_int(rng, 256, 16_384), steps=rng.randint(1, 10))
    if kind in ("loss_grad", "density"):
        return dict(kind=kind, n=_log_int(rng, 500, 200_000))
    if kind == "sample":
        return dict(kind=kind, n=_log_int(rng, 1000, 2_000_000))
    return dict(kind=kind, n=_log_int(rng, 5000, 1_000_000))


def work(case):
    kind = case["kind"]
    if kind in ("integrate", "proceed"):
        cfg = W.config(case["workload"])
        grid = 8.0 * cfg["ndim"] * (cfg["nbins"] + 1)
        return {"bytes": 2.0 * grid, "flops": FLOPS_EVENT[case["workload"]] * case["n"] * case["iters"]}
    if kind == "schedule":
        cfg = W.config(case["workload"])
        n = case["n1"] * case["k1"] + case["n2"] * case["k2"]
        return {"bytes": 16.0 * cfg["ndim"] * (cfg["nbins"] + 1), "flops": FLOPS_EVENT[case["workload"]] * n}
    if kind == "grad":
        return {"bytes": 8.0 * 16 * case["points"], "flops": (200.0 + FLOPS_GRAD_POINT * case["points"]) * case["n"]}
    n = case["n"]
    if kind == "train":
        per = 3.0 * FLOPS_FLOW_EVENT * case["batch"]
        return {"bytes": case["steps"] * (40.0 * case["batch"] + 24.0 * F.NPARAMS), "flops": case["steps"] * per}
    if kind == "loss_grad":
        return {"bytes": 40.0 * n + 8.0 * F.NPARAMS, "flops": 3.0 * FLOPS_FLOW_EVENT * n}
    if kind == "density":
        return {"bytes": 36.0 * n + 4.0 * F.NPARAMS, "flops": FLOPS_FLOW_EVENT * n}
    if kind == "sample":
        return {"bytes": 68.0 * n + 4.0 * F.NPARAMS, "flops": FLOPS_FLOW_EVENT * n}
    return {"bytes": 4.0 * F.NPARAMS + 16.0 * 8 * 101, "flops": (FLOPS_FLOW_EVENT + FLOPS_EVENT["ww_4l"]) * n}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
OBS_RANGE = {"dy_z": (81.0, 101.0), "w_plus": (20.0, 70.0), "ww_4l": (60.0, 100.0), "ww_had": (60.0, 100.0)}


def _integrator(case, seed, n):
    cfg = W.config(case["workload"])
    return P.Integrator(cfg["process"], cfg["ndim"], cfg["nbins"], 1 + seed, cfg["alpha"], cfg["params"],
                        precision=P.FP32_ME if case.get("fp32") else P.FP64, max_events=n)


def _adapted(g):
    for _ in range(GRID_ADAPT[0]):
        g.iterate(GRID_ADAPT[1], sync=False)
        g.refine()
    return g.get_state()


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(1000 + seed)


def _theta(seed, spread=0.3):
    """Parameters of a proposal some way into its training: He-uniform hidden layers and
    an output layer whose spline parameters have a spread of a few tenths (more while
    it is still far from the data, as in the training cases)."""
    g = _generator(seed)
    parts = []
    for _ in range(6):
        for fan, size in ((4, 4 * 128), (0, 128), (128, 128 * 128), (0, 128)):
            u = torch.rand(size, generator=g, device="cuda") * 2 - 1
            parts.append(u * (math.sqrt(6 / fan) if fan else 0.05))
        parts.append(torch.randn(128 * 188, generator=g, device="cuda") * (spread / math.sqrt(128)))
        parts.append(torch.randn(188, generator=g, device="cuda") * 0.05)
    return torch.cat(parts)


def _points(n, seed):
    """Weighted events: uniform points of the unit cube (as an iteration on an adapted grid
    has them) and positive weights with the correlations and the spread (relative variance
    about 0.4) that the grid leaves behind."""
    g = _generator(seed + 77)
    y = torch.rand(n, 8, generator=g, device="cuda")
    z = y.double()
    s = torch.sin(3 * z[:, 0] * z[:, 1]) + torch.cos(4 * (z[:, 2] - z[:, 5])) + z[:, 3] * (1 - z[:, 6]) - z[:, 4] * z[:, 7]
    return y, 10.0 * torch.exp(0.7 * s)


def _adjoint_theta(points, seed):
    return torch.tensor(W.adjoint_points(points, 2 + seed), device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "seed": seed}
    if kind == "proceed":
        g = s["g"] = _integrator(case, seed, max(case["n"], GRID_ADAPT[1]))
        s["start"] = _adapted(g)
        if case["strata"]:
            g.set_strata(case["strata"])
            g.set_strata_beta(case["beta"])
    elif kind == "schedule":
        s["g"] = _integrator(case, seed, max(case["n1"], case["n2"]))
        s["start"] = s["g"].get_state()
        s["sizes"] = [case["n1"]] * case["k1"] + [case["n2"]] * case["k2"]
    elif kind == "grad":
        g = s["g"] = _integrator({"workload": "dy_z"}, seed, GRID_ADAPT[1])
        _adapted(g)
        s["theta"] = _adjoint_theta(case["points"], seed).requires_grad_(True)
        s["upstream"] = 1.0 + 0.25 * torch.rand(case["points"], generator=_generator(seed), device="cuda", dtype=torch.float64)
    elif kind == "train":
        s["flow"] = P.Flow(max_batch=case["batch"], seed=1 + seed)
        s["theta"] = _theta(seed, 0.6)
        s["y"], s["w"] = _points(case["n"], seed)
    elif kind in ("loss_grad", "density", "sample"):
        s["flow"] = P.Flow(max_batch=1 if kind == "sample" else min(case["n"], BATCH_MAX), seed=1 + seed)
        s["flow"].set_params(_theta(seed))
        s["y"], s["w"] = _points(case["n"], seed)
    elif kind == "flow_iterate":
        g = s["g"] = _integrator({"workload": "ww_4l"}, seed, max(case["n"], GRID_ADAPT[1]))
        s["start"] = _adapted(g)
        s["flow"] = P.Flow(max_batch=1, max_sample=case["n"], seed=1 + seed)
        s["flow"].set_params(_theta(seed))
    return s


# ---------------------------------------------------------------------------
# a pass
# ---------------------------------------------------------------------------
def _iterations(g, sizes, read):
    """Iterations and refinements; with read the program looks at each one's estimate."""
    seen = []
    for n in sizes:
        r = g.iterate(n, sync=read)
        g.refine()
        if read:
            seen.append(r)
    return seen


def _summary(g, seen):
    r = g.result()
    d, sums = g.get_hist()
    out = {"result": np.array([r["I"], r["sigma"], r["chi2_dof"]]), "grid": g.get_grid(), "hist": d, "sums": sums}
    if seen:
        out["each"] = np.array([[x["I"], x["var"]] for x in seen])
        out["counts"] = np.array([[x["n_events"], x["n_nonzero"], x["n_nonfinite"]] for x in seen])
    return out


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "integrate":
        g = _integrator(case, state["seed"], case["n"])
        if case["obs"]:
            g.set_observable(case["obs"], *OBS_RANGE[case["workload"]])
        seen = _iterations(g, [case["n"]] * case["iters"], case["read"])
        out = _summary(g, seen)
        if case["obs"]:
            out["obs"] = np.stack(g.get_observable())
        g.close()
        return out
    if kind == "proceed":
        g = state["g"]
        g.set_state(state["start"])
        return _summary(g, _iterations(g, [case["n"]] * case["iters"], case["read"]))
    if kind == "schedule":
        g = state["g"]
        g.set_state(state["start"])
        g.run_schedule(state["sizes"])
        late = g.result(first=case["k1"])
        return dict(_summary(g, None), late=np.array([late["I"], late["sigma"], late["chi2_dof"]]))
    if kind == "grad":
        theta = state["theta"]
        theta.grad = None
        sigma = P.vegas_sigma(theta, state["g"], case["n"], GRID_ADAPT[0])
        sigma.backward(state["upstream"])
        return {"sigma": sigma.detach(), "grad": theta.grad}
    flow = state["flow"]
    if kind == "train":
        flow.set_params(state["theta"])
        for _ in range(case["steps"] - 1):
            flow.train_step(state["y"], state["w"], case["batch"])
        loss = flow.train_step(state["y"], state["w"], case["batch"], with_loss=True)
        return {"loss": loss, "theta": flow.get_params()}
    if kind == "loss_grad":
        loss, grad = flow.loss_grad(state["y"], state["w"])
        return {"loss": loss, "grad": grad}
    if kind == "density":
        return {"logq": flow.density(state["y"])}
    if kind == "sample":
        y, logq = flow.sample(state["y"])
        return {"y": y, "logq": logq}
    g = state["g"]
    g.set_state(state["start"])
    r = g.iterate_flow(flow, case["n"])
    d, sums = g.get_hist()
    return {"each": np.array([r["I"], r["var"]]), "counts": np.array([r["n_events"], r["n_nonzero"], r["n_nonfinite"]]),
            "hist": d, "sums": sums}


# ---------------------------------------------------------------------------
# the same results from plain binary64 PyTorch
# ---------------------------------------------------------------------------
DEVICE = "cuda" if torch.cuda.is_available() else "cpu"
CHUNK = 1 << 20
M32 = 0xFFFFFFFF


def _uniforms(seed, iteration, first, n, ndim):
    """[ndim][n] uniforms of events first .. first + n: Philox4x32-10, counter (event,
    iteration, call), key seed; words (1:0) and (3:2) of a call give two uniforms."""
    ev = torch.arange(first, first + n, device=DEVICE)
    u = []
    for call in range((ndim + 1) // 2):
        c = [ev & M32, ev >> 32, torch.full_like(ev, iteration), torch.full_like(ev, call)]
        k0, k1 = seed & M32, seed >> 32
        for _ in range(10):
            p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57  # the low 64 bits: both halves
            c = [((p1 >> 32) & M32) ^ c[1] ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c[3] ^ k1, p0 & M32]
            k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
        for lo, hi in ((c[0], c[1]), (c[2], c[3])):
            u.append(((hi << 20 | lo >> 12).double() + 0.5) * 2.0 ** -52)
    return torch.stack(u[:ndim])


_NAMES = ("alpha", "sw2", "mz", "gz", "mw", "gw", "rs", "A", "a", "b", "mlo", "mhi", "ptmin", "etamax", "vud", "conv")


def _physics(workload):
    return dict(zip(_NAMES, (float(v) for v in W.config(workload)["params"])))


def _bw(M, G, lo2, hi2, x):
    """Breit-Wigner map of x onto m^2 in [lo2, hi2] (below the pole from the lower edge, by
    the tangent's addition theorem) and dm^2/dx."""
    MG, tlo = M * G, (lo2 - M * M) / (M * G)
    rho_lo = math.atan(tlo)
    rng = (torch.atan((hi2 - M * M) / MG) if torch.is_tensor(hi2) else math.atan((hi2 - M * M) / MG)) - rho_lo
    rho, t = rho_lo + x * rng, torch.tan(x * rng)
    m2 = torch.where(rho < 0, lo2 + MG * (1 + tlo * tlo) * t / (1 - tlo * t), M * M + MG * torch.tan(rho))
    return m2, rng * ((m2 - M * M) ** 2 + MG * MG) / MG


def _parton(q, lnx):
    return q["A"] * torch.exp(q["a"] * lnx) * (-torch.expm1(lnx)) ** q["b"]


def _couplings(sw2, flavour):
    """(Q, g_L, g_R) of u (0), d (1) or a charged lepton (2)."""
    T3, Q = ((0.5, 2 / 3), (-0.5, -1 / 3), (-0.5, -1.0))[flavour]
    sc = (sw2 * (1 - sw2)) ** 0.5
    return Q, (T3 - Q * sw2) / sc, -Q * sw2 / sc


def _dy_kinematics(q, x):
    """m^2, ln x1, ln x2, cos theta and the phase-space factor with the flux."""
    m2, jbw = _bw(q["mz"], q["gz"], q["mlo"] ** 2, q["mhi"] ** 2, x[0])
    L = torch.log(m2 / q["rs"] ** 2)
    l1 = x[1] * L
    c = 2 * x[2] - 1
    return m2, l1, L - l1, c, q["conv"] * jbw * (-L / q["rs"] ** 2) * 2 / (2 * m2) / (16 * math.pi)


def _dy_me2(q, m2, c):
    """sum over u, d, both beam orderings and helicities, averaged; q's entries may be
    tensors that broadcast against the events."""
    e2 = 4 * math.pi * q["alpha"]
    ds, mg = m2 - q["mz"] ** 2, q["mz"] * q["gz"]
    pre, pim = ds / (ds * ds + mg * mg), -mg / (ds * ds + mg * mg)
    total = 0.0
    gl = _couplings(q["sw2"], 2)
    for f in (0, 1):
        gq = _couplings(q["sw2"], f)
        for h in (1, 2):
            for hp in (1, 2):
                g = gq[h] * gl[hp]
                amp2 = (-gq[0] / m2 + g * pre) ** 2 + (g * pim) ** 2
                total = total + amp2 * ((1 + c) ** 2 + (1 - c) ** 2)
    return e2 * e2 * m2 * m2 * total / 12


def _f_dy(q, x):
    m2, l1, l2, c, ps = _dy_kinematics(q, x)
    return ps * _parton(q, l1) * _parton(q, l2) * _dy_me2(q, m2, c), torch.sqrt(m2)


def _f_w(q, x):
    hi = q["mhi"] if q["mhi"] > 0 else q["rs"]
    m2, jbw = _bw(q["mw"], q["gw"], q["mlo"] ** 2, hi * hi, x[0])
    L = torch.log(m2 / q["rs"] ** 2)
    l1 = x[1] * L
    l2 = L - l1
    c = 2 * x[2] - 1
    pt = 0.5 * torch.sqrt(m2 * (1 - c) * (1 + c))
    x1, x2 = torch.exp(l1), torch.exp(l2)
    beta = (x1 - x2) / (x1 + x2)
    cos_lab = (c + beta) / (1 + beta * c)
    ok = (pt > q["ptmin"]) & (cos_lab.abs() < math.tanh(q["etamax"]))
    g2 = 4 * math.pi * q["alpha"] / q["sw2"]
    den = (m2 - q["mw"] ** 2) ** 2 + (q["mw"] * q["gw"]) ** 2
    me = g2 * g2 * q["vud"] ** 2 * (m2 / 2) ** 2 * ((1 - c) ** 2 + (1 + c) ** 2) / (12 * den)
    w = q["conv"] * jbw * (-L / q["rs"] ** 2) / (2 * m2) / (8 * math.pi) * _parton(q, l1) * _parton(q, l2) * me
    return torch.where(ok, w, 0.0), pt


def _direction(xc, xf):
    c, f = 2 * xc - 1, 2 * math.pi * xf
    s = torch.sqrt((1 - c) * (1 + c))
    return [s * torch.cos(f), s * torch.sin(f), c]


def _decay(Q, m, n):
    """Massless two-body decay of Q (mass m) along n in its rest frame: both momenta."""
    out = []
    for sign in (1.0, -1.0):
        k = [0.5 * m] + [sign * 0.5 * m * v for v in n]
        E = (Q[0] * k[0] + Q[1] * k[1] + Q[2] * k[2] + Q[3] * k[3]) / m
        f = (k[0] + E) / (Q[0] + m)
        out.append([E] + [k[i] + f * Q[i] for i in (1, 2, 3)])
    return out


def _weyl(p):
    """Left-handed massless two-spinor of p (its phase is free)."""
    up = p[3] >= 0
    r = torch.sqrt(p[0] + p[3].abs())
    z = torch.complex(p[1], p[2]) / r
    return torch.where(up, -z.conj(), -r.to(z.dtype)), torch.where(up, r.to(z.dtype), z)


def _current(p, k):
    """a^dagger sigma-bar^mu b for the spinors of p and k."""
    (a0, a1), (b0, b1) = _weyl(p), _weyl(k)
    a0, a1 = a0.conj(), a1.conj()
    return [a0 * b0 + a1 * b1, -(a0 * b1 + a1 * b0), 1j * (a0 * b1 - a1 * b0), a1 * b1 - a0 * b0]


def _mdot(a, b):
    return a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3]


def _f_ww(q, x, rs=None):
    """q qbar -> W+ W- -> e+ nu mu- nubar at sqrt(shat) = rs, doubly resonant diagrams."""
    rs = q["rs"] + 0 * x[0] if rs is None else rs
    sh = rs * rs
    MW, GW = q["mw"], q["gw"]
    mp2, jp = _bw(MW, GW, 0.0, sh, x[0])
    mp = torch.sqrt(mp2.clamp_min(0))
    mm2, jm = _bw(MW, GW, 0.0, (rs - mp) ** 2, x[1])
    mm = torch.sqrt(mm2.clamp_min(0))
    lam = (sh - mp2 - mm2) ** 2 - 4 * mp2 * mm2
    ok = (mp2 > 0) & (mm2 > 0) & (lam > 0)
    sl = torch.sqrt(lam.clamp_min(0))
    k, n = sl / (2 * rs), _direction(x[2], x[3])
    qp = [(sh + mp2 - mm2) / (2 * rs)] + [k * v for v in n]
    qm = [(sh - mp2 + mm2) / (2 * rs)] + [-k * v for v in n]
    l3, l4 = _decay(qp, mp, _direction(x[4], x[5]))
    l5, l6 = _decay(qm, mm, _direction(x[6], x[7]))
    e2 = 4 * math.pi * q["alpha"]
    g2 = e2 / q["sw2"]
    ep = [math.sqrt(g2 / 2) * v / torch.complex(mp2 - MW * MW, MW * GW + 0 * mp2) for v in _current(l4, l3)]
    em = [math.sqrt(g2 / 2) * v / torch.complex(mm2 - MW * MW, MW * GW + 0 * mm2) for v in _current(l5, l6)]
    a1 = _mdot([2 * qp[i] + qm[i] for i in range(4)], em)
    a2 = _mdot(ep, em)
    a3 = _mdot([qp[i] + 2 * qm[i] for i in range(4)], ep)
    V1, V2 = (ep[i] * a1 + a2 * (qm[i] - qp[i]) - em[i] * a3 for i in (1, 2))
    jV = {0: -rs * (V1 - 1j * V2), 1: -rs * (V1 + 1j * V2)}
    prop = 1 / torch.complex(sh - q["mz"] ** 2, q["mz"] * q["gz"] + 0 * sh)
    cot = math.sqrt((1 - q["sw2"]) / q["sw2"])
    me2 = 0.0
    for flavour in (0, 1):
        Q, gL, gR = _couplings(q["sw2"], flavour)
        for h, gz in ((0, gL), (1, gR)):
            amp = e2 * (Q / sh + gz * cot * prop) * jV[h]
            if h == 0:  # the exchange diagram: the boson next to the incoming quark first
                one, two, out = (ep, em, qp) if flavour == 0 else (em, ep, qm)
                kk = [0.5 * rs - out[0], -out[1], -out[2], 0.5 * rs - out[3]]
                c01, c11 = one[1] - 1j * one[2], one[0] - one[3]
                y0 = (kk[0] - kk[3]) * c01 - torch.complex(kk[1], -kk[2]) * c11
                y1 = -torch.complex(kk[1], kk[2]) * c01 + (kk[0] + kk[3]) * c11
                chain = (two[0] + two[3]) * y0 + (two[1] - 1j * two[2]) * y1
                amp = amp + 0.5 * g2 * rs * chain / _mdot(kk, kk)
            me2 = me2 + amp.real ** 2 + amp.imag ** 2
    ps = sl / (8 * math.pi * sh) * jp * jm / (4 * math.pi ** 2) / (64 * math.pi ** 2)
    return torch.where(ok, q["conv"] / (2 * sh) / 12 * me2 * ps, 0.0), torch.where(mp2 > 0, mp, 0.0)


def _f_ww_had(q, x):
    S, hi = q["rs"] ** 2, q["mhi"] if q["mhi"] > 0 else q["rs"]
    Llo, Lhi = math.log(q["mlo"] ** 2 / S), math.log(hi * hi / S)
    L = Lhi + x[8] * (Llo - Lhi)
    tau, l1 = torch.exp(L), x[9] * L
    w, o = _f_ww(q, x, torch.sqrt(tau * S))
    return 2 * tau * (Lhi - Llo) * (-L) * _parton(q, l1) * _parton(q, L - l1) * w, o


INTEGRAND = {"dy_z": _f_dy, "w_plus": _f_w, "ww_4l": _f_ww, "ww_had": _f_ww_had}


class _Vegas:
    """The method in binary64: iterations, the refinement, the combinations."""

    def __init__(self, workload, seed, obs=0):
        cfg = W.config(workload)
        self.f, self.q, self.seed = INTEGRAND[workload], _physics(workload), 1 + seed
        self.D, self.n, self.alpha = cfg["ndim"], cfg["nbins"], cfg["alpha"]
        self.edges = (torch.arange(self.n + 1, device=DEVICE).double() / self.n).repeat(self.D, 1)
        self.j, self.history, self.sig = 0, [], None
        self.nobs, self.range, self.obs_history = obs, OBS_RANGE[workload], []

    def map(self, u):
        """Grid map of uniforms u [D][N]: points, Jacobian, bins."""
        t = u * self.n
        k = t.long().clamp_max(self.n - 1)
        lo, hi = torch.gather(self.edges, 1, k), torch.gather(self.edges, 1, k + 1)
        return lo + (t - k) * (hi - lo), (self.n * (hi - lo)).prod(0), k

    def counts(self, n, H, beta):
        """Events per hypercube of an adaptive iteration."""
        p = self.sig ** beta if self.sig is not None else torch.ones(H, dtype=torch.float64, device=DEVICE)
        free, total = n - 2 * H, p.sum()
        c = torch.floor(free * p / total).long() if total > 0 else torch.full((H,), n, device=DEVICE)
        if int(c.sum()) > free:
            c = torch.full((H,), free // H, device=DEVICE)
        return c + 2 + (torch.arange(H, device=DEVICE) < free - int(c.sum()))

    def iterate(self, n, m=0, beta=0.0, proposal=None):
        H = m ** self.D if m else 0
        cnt = self.counts(n, H, beta) if H and beta else torch.full((H,), n // H, device=DEVICE) if H else None
        n = int(cnt.sum()) if H else n
        cube = torch.repeat_interleave(torch.arange(H, device=DEVICE), cnt) if H else None
        d = torch.zeros(self.D * self.n, dtype=torch.float64, device=DEVICE)
        ob = torch.zeros(2, self.nobs + 2, dtype=torch.float64, device=DEVICE)
        ws, off = [], torch.arange(self.D, device=DEVICE)[:, None] * self.n
        for first in range(0, n, CHUNK):
            k = min(CHUNK, n - first)
            u = _uniforms(self.seed, self.j, first, k, self.D)
            lq = 0.0
            if H:
                h = cube[first:first + k]
                u = torch.stack([((h // m ** a) % m + u[a]) / m for a in range(self.D)])
            if proposal is not None:
                y, lq = proposal(u.t().float().double())
                u = y.t().contiguous().clamp(2.0 ** -40, 1 - 2.0 ** -40)
            x, J, bins = self.map(u)
            w, o = self.f(self.q, x)
            w = w * J * (torch.exp(-lq) if proposal is not None else 1.0)
            if H and beta:
                w = w * (n / (H * cnt[h].double()))
            w = torch.where(torch.isfinite(w * w), w, 0.0)
            d.index_add_(0, (bins + off).reshape(-1), (w * w).repeat(self.D))
            if self.nobs:
                lo, hi = self.range
                b = torch.floor((o - lo) * (self.nobs / (hi - lo))).clamp(-1, self.nobs).long() + 1
                b = torch.where(o < lo, 0, torch.where(o < hi, b.clamp_max(self.nobs), self.nobs + 1))
                ob[0].index_add_(0, b, w)
                ob[1].index_add_(0, b, w * w)
            ws.append(w)
        w = torch.cat(ws)
        self.d, self.s1, self.s2 = d, float(w.sum()), float((w * w).sum())
        I = self.s1 / n
        if H:
            c = cnt.double()
            zero = torch.zeros(H, dtype=torch.float64, device=DEVICE)
            mean = zero.index_add(0, cube, w) / c
            V = zero.index_add(0, cube, (w - mean[cube]) ** 2) / (c - 1)
            var = float((c * V).sum()) / (n * n)  # equal counts: n = H c
            self.sig = torch.sqrt(V) / (n / (H * c))
        else:
            var = float(((w - I) ** 2).sum()) / n / (n - 1)
        if self.nobs:
            h = ob[0] / n
            self.obs_history.append((h, (ob[1] / n - h * h) / (n - 1)))
        self.history.append((I, var))
        self.j += 1
        return I, var

    def refine(self):
        n = self.n
        for a in range(self.D):
            d = self.d[a * n:(a + 1) * n].cpu().numpy()
            if not d.sum() > 0:
                continue
            s = np.empty(n)
            s[1:-1] = (d[:-2] + d[1:-1] + d[2:]) / 3
            s[0], s[-1] = (d[0] + d[1]) / 2, (d[-2] + d[-1]) / 2
            r = s / s.sum()
            with np.errstate(divide="ignore", invalid="ignore"):
                m = np.where(r == 0, 0.0, np.where(r == 1, 1.0, ((r - 1) / np.log(r)) ** self.alpha))
            cm = np.concatenate([[0.0], np.cumsum(m)])
            e, t = self.edges[a].cpu().numpy(), np.arange(1, n) * (cm[-1] / n)
            j = np.clip(np.searchsorted(cm, t, side="left") - 1, 0, n - 1)
            f = np.clip((t - cm[j]) / m[j], 0.0, 1.0)
            new = np.concatenate([[0.0], e[j] + f * (e[j + 1] - e[j]), [1.0]])
            self.edges[a] = torch.from_numpy(new).to(DEVICE)

    def combined(self, first=0):
        I, v = np.array(self.history[first:]).T
        mean = (I / v).sum() / (1 / v).sum()
        chi = ((I - mean) ** 2 / v).sum()
        return np.array([mean, (1 / v).sum() ** -0.5, chi / (len(I) - 1) if len(I) > 1 else 0.0])

    def summary(self, each):
        out = {"result": self.combined(), "grid": self.edges.cpu().numpy(),
               "hist": self.d.view(self.D, self.n).cpu().numpy(), "sums": np.array([self.s1, self.s2])}
        if each:
            out["each"], out["counts"] = np.array(each), None
        if self.nobs:
            wj = torch.tensor([1 / v for _, v in self.history], dtype=torch.float64, device=DEVICE)[:, None]
            h, v = (torch.stack(t) for t in zip(*self.obs_history))
            comb, err = (wj * h).sum(0) / wj.sum(), torch.sqrt((wj * wj * v).sum(0)) / wj.sum()
            out["obs"] = torch.stack([h[-1], torch.sqrt(v[-1].clamp_min(0)), comb, err]).cpu().numpy()
        return out

    def adapt(self):
        for _ in range(GRID_ADAPT[0]):
            self.iterate(GRID_ADAPT[1])
            self.refine()
        return self


LAYERS = ((4, 5, 6, 7), (0, 1, 2, 3), (1, 3, 5, 7), (0, 2, 4, 6), (2, 3, 6, 7), (0, 1, 4, 5))  # transformed
EPS = 1e-3
SHIFT = math.log(math.expm1(1 - EPS))


def _flow(v, theta, inverse):
    """The coupling-layer flow in binary64: (z, log q) of points y, or (y, log q) of z."""
    out, logq, size = list(v.unbind(1)), 0.0, F.NPARAMS // 6
    for l in (range(5, -1, -1) if inverse else range(6)):
        W1, b1, W2, b2, W3, b3 = torch.split(theta[l * size:(l + 1) * size], [512, 128, 16384, 128, 24064, 188])
        cond = torch.stack([out[a] for a in range(8) if a not in LAYERS[l]], 1)
        h = torch.relu(torch.relu(cond @ W1.view(4, 128) + b1) @ W2.view(128, 128) + b2)
        raw = (h @ W3.view(128, 188) + b3).view(-1, 4, 47)
        one = torch.ones_like(raw[..., :1])
        knots = []
        for r in (raw[..., :16], raw[..., 16:32]):
            inner = torch.cumsum(EPS + (1 - 16 * EPS) * torch.softmax(r, -1), -1)[..., :-1]
            knots.append(torch.cat([0 * one, inner, one], -1))
        xk, yk = knots
        dk = torch.cat([one, EPS + torch.nn.functional.softplus(raw[..., 32:] + SHIFT), one], -1)
        p = torch.stack([out[a] for a in LAYERS[l]], 1)[..., None]
        k = ((yk if inverse else xk)[..., 1:-1] < p).sum(-1, keepdim=True)
        x0, x1, y0, y1, d0, d1 = (torch.gather(t, -1, k + i) for t in (xk, yk, dk) for i in (0, 1))
        w, hh = x1 - x0, y1 - y0
        s = hh / w
        g = d1 + d0 - 2 * s
        if inverse:
            dy = p - y0
            a, b, c = hh * (s - d0) + dy * g, hh * d0 - dy * g, -s * dy
            xi = (2 * c / (-b - torch.sqrt((b * b - 4 * a * c).clamp_min(0)))).clamp(0, 1)
            q = x0 + xi * w
        else:
            xi = (p - x0) / w
            q = y0 + hh * (s * xi * xi + d0 * xi * (1 - xi)) / (s + g * xi * (1 - xi))
        t = xi * (1 - xi)
        slope = s * s * (d1 * xi * xi + 2 * s * t + d0 * (1 - xi) ** 2) / (s + g * t) ** 2
        logq = logq + torch.log(slope).sum((1, 2))
        for i, a in enumerate(LAYERS[l]):
            out[a] = q[:, i, 0]
    return torch.stack(out, 1), logq


def _flow_chunks(v, theta, inverse, chunk=1 << 16):
    parts = [_flow(v[i:i + chunk], theta, inverse) for i in range(0, v.shape[0], chunk)]
    return torch.cat([a for a, _ in parts]), torch.cat([b for _, b in parts])


def _flow_loss(theta, y, w, chunk=1 << 14):
    """L = -sum w log q / sum w and its gradient."""
    t = theta.clone().requires_grad_(True)
    total, loss = w.sum(), 0.0
    for i in range(0, y.shape[0], chunk):
        part = -(w[i:i + chunk] * _flow(y[i:i + chunk], t, False)[1]).sum() / total
        part.backward()
        loss += float(part.detach())
    return loss, t.grad


def _batch(n, batch, step):
    """Indices of a training step's batch: the epoch's bijection i -> (a i + c) mod n."""
    per = -(-n // batch)
    epoch = step // per
    s0, s1 = (epoch * 0x9E3779B9 + 0x7F4A7C15) & M32, (epoch >> 32) ^ 0x85EBCA6B
    for r in range(3):
        s0 ^= (s1 * 0xC2B2AE35 + r) & M32
        s1 ^= ((s0 << 13) | (s0 >> 19)) & M32
    a, c = (s0 | 1) % n or 1, s1 % n
    while math.gcd(a, n) != 1:
        a = (a + 2) % n or 1
    i = ((step % per) * batch + torch.arange(batch, device=DEVICE)) % n
    return (a * i + c) % n


def _exact_grad(case, seed):
    v = _Vegas("dy_z", seed).adapt()
    q, n = v.q, case["n"]
    theta = _adjoint_theta(case["points"], seed).requires_grad_(True)
    sigma = 0.0
    for first in range(0, n, 1 << 15):
        k = min(1 << 15, n - first)
        x, J, _ = v.map(_uniforms(v.seed, v.j, first, k, 3))
        m2, l1, l2, c, ps = _dy_kinematics(q, x)
        mz, gz, sw2, a, b = (t[:, None] for t in theta.unbind(1))
        me = _dy_me2(dict(q, mz=mz, gz=gz, sw2=sw2), m2, c)
        ff = q["A"] ** 2 * torch.exp(a * (l1 + l2) + b * torch.log(torch.expm1(l1) * torch.expm1(l2)))
        part = (J * ps * ff * me).sum(1) / n
        part.backward(1.0 + 0.25 * torch.rand(case["points"], generator=_generator(seed), device="cuda", dtype=torch.float64))
        sigma = sigma + part.detach()
    return {"sigma": sigma, "grad": theta.grad}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("integrate", "proceed"):
        v = _Vegas(case["workload"], seed, case.get("obs", 0))
        if kind == "proceed":
            v.adapt()
        each = []
        for _ in range(case["iters"]):
            each.append(v.iterate(case["n"], case["strata"], case["beta"]))
            v.refine()
        return v.summary(each if case["read"] else None)
    if kind == "schedule":
        v = _Vegas(case["workload"], seed)
        for n in [case["n1"]] * case["k1"] + [case["n2"]] * case["k2"]:
            v.iterate(n)
            v.refine()
        return dict(v.summary(None), late=v.combined(case["k1"]))
    if kind == "grad":
        return _exact_grad(case, seed)
    theta = _theta(seed, 0.6 if kind == "train" else 0.3).double()
    if kind == "flow_iterate":
        v = _Vegas("ww_4l", seed).adapt()
        each = v.iterate(case["n"], proposal=lambda z: _flow_chunks(z, theta, True))
        s = v.summary([each])
        # a histogram bin's sum of w^2 hangs on its few largest events, whose 1 / q^2
        # carries the 16-bit rounding of the library's proposal: no value to hold it to
        return {"each": s["each"][0], "counts": None, "hist": None, "sums": s["sums"]}
    y, w = _points(case["n"], seed)
    y = y.double()
    if kind == "density":
        return {"logq": _flow_chunks(y, theta, False)[1]}
    if kind == "sample":
        a, lq = _flow_chunks(y, theta, True)
        return {"y": a, "logq": lq}
    if kind == "loss_grad":
        loss, grad = _flow_loss(theta, y, w)
        return {"loss": loss, "grad": grad}
    m1, m2 = torch.zeros_like(theta), torch.zeros_like(theta)
    for s in range(case["steps"]):
        i = _batch(case["n"], case["batch"], s)
        loss, g = _flow_loss(theta, y[i], w[i])
        m1, m2 = 0.9 * m1 + 0.1 * g, 0.999 * m2 + 0.001 * g * g
        theta = theta - 1e-3 * (m1 / (1 - 0.9 ** (s + 1))) / (torch.sqrt(m2 / (1 - 0.999 ** (s + 1))) + 1e-8)
    return {"loss": loss, "theta": theta}
