"""Workloads of the batched ODE integrators, through the package's public entry points.

A pass is one integration (or gradient) of a whole batch, as an operator-split
simulation calls it once per global step.  The listed cases are the
configurations of inputs.WORKLOADS and of the ragged batch at sizes one pass
takes from under a millisecond to about a second, plus small and odd batches;
draw() spreads the same kinds over the same ranges of sizes.

Kinds:
  vdp        van der Pol oscillators, RKCK (nonstiff) or RKC (stiff, 10-60 stages)
  net        isothermal mass-action networks of 9, 13, 32 or 53 species
  thermal    the networks with the energy equation (state T, Y)
  pleiades   the seven-body problem, ten restart global steps
  solve      forward and backward of rkc_solve / rkck_solve (dL/dy0, dL/dlnA)
  ragged     the four networks in one batch over operator-splitting substeps
"""
import functools
import math

import numpy as np
import torch

import paper_1611_02274_amd as rk
from paper_1611_02274_amd import flops, inputs

RTOL, ATOL = 1e-8, 1e-12            # the networks' tolerances


def listed():
    return [
        # a small batch of cheap systems: latency of one wave's steps and of the call
        dict(name="vdp_rkck_4096", kind="vdp", method="rkck", n=4096, t1=10.0, schedule=1),
        # stiff oscillators: long stage recursions, odd size, the automatic schedule
        dict(name="vdp_rkc_stiff_5003", kind="vdp", method="rkc", n=5003, t1=1.0, schedule=0),
        # a few hundred cells of a small reduced mechanism per operator-splitting step
        dict(name="net9_rkc_300", kind="net", species=9, method="rkc", n=300, schedule=0,
             cost_order=0),
        # the 13-species batch in its tuned launch
        dict(name="net13_rkc_262144", kind="net", species=13, method="rkc", n=262144, schedule=1,
             cost_order=1),
        # a mid-sized batch of a mid-sized mechanism, not a multiple of any tile
        dict(name="net32_rkc_16411", kind="net", species=32, method="rkc", n=16411, schedule=0,
             cost_order=0),
        # the largest mechanism under both methods: the bulk of a chemistry step
        dict(name="net53_rkck_65536", kind="net", species=53, method="rkck", n=65536, schedule=0,
             cost_order=0),
        dict(name="net53_rkc_65536", kind="net", species=53, method="rkc", n=65536, schedule=0,
             cost_order=0),
        # energy equation: the small network, one global step in its tuned launch
        dict(name="net13_thermal_rkc_65536", kind="thermal", species=13, method="rkc", n=65536,
             schedule=1, cost_order=1),
        # energy equation: the largest network
        dict(name="net53_thermal_rkc_8191", kind="thermal", species=53, method="rkc", n=8191,
             schedule=3, cost_order=0),
        # nonstiff few-body problem at tight tolerance
        dict(name="pleiades_rkck_262144", kind="pleiades", method="rkck", n=262144, steps=10),
        # parameter fitting: forward with tape, reverse sweep, shared ln A gradient
        dict(name="net13_solve_rkc_65536", kind="solve", species=13, method="rkc", n=65536),
        # mechanisms of different sizes in one batch, two substeps in a captured graph
        dict(name="ragged_50000", kind="ragged", n=50000, substeps=2, graph=True),
    ]


def _size(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return n | 1 if rng.random() < 0.6 else n


def draw(rng):
    kind = rng.choice(["vdp", "net", "net", "net", "net", "thermal", "pleiades", "solve",
                       "ragged"])
    if kind == "vdp":
        if rng.random() < 0.5:
            return dict(kind=kind, method="rkck", n=_size(rng, 64, 65536), t1=10.0,
                        schedule=rng.choice([0, 1]))
        return dict(kind=kind, method="rkc", n=_size(rng, 64, 16384), t1=1.0,
                    schedule=rng.choice([0, 1]))
    if kind == "net":
        sp = rng.choice([9, 13, 32, 53])
        small = sp <= 13
        return dict(kind=kind, species=sp, method=rng.choice(["rkc", "rkck"]),
                    n=_size(rng, 200, 262144 if small else 49152),
                    schedule=rng.choice([0, 1, 2]) if small else rng.choice([0, 3]),
                    cost_order=rng.choice([0, 1]) if small else 0)
    if kind == "thermal":
        sp = rng.choice([9, 13, 32, 53])
        small = sp <= 13
        return dict(kind=kind, species=sp, method="rkc",
                    n=_size(rng, 200, 65536 if small else 8192),
                    schedule=rng.choice([0, 1]) if small else rng.choice([0, 3]),
                    cost_order=rng.choice([0, 1]) if small else 0)
    if kind == "pleiades":
        return dict(kind=kind, method="rkck", n=_size(rng, 500, 262144), steps=10)
    if kind == "solve":
        return dict(kind=kind, species=rng.choice([9, 13]), method=rng.choice(["rkc", "rkck"]),
                    n=_size(rng, 500, 65536))
    return dict(kind="ragged", n=_size(rng, 2000, 50000), substeps=rng.choice([1, 2]),
                graph=rng.choice([True, False]))


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=None)
def _network(species, thermal=False):
    return inputs.thermal_network(species) if thermal else inputs.standard_network(species)


def _t_range(species):
    return (900.0, 2800.0) if species >= 32 else (1000.0, 2500.0)


def _interval(case):
    """(t0, t1, rtol, atol) of one pass."""
    if case["kind"] == "vdp":
        return (0.0, case["t1"], 1e-8, 1e-10) if case["method"] == "rkck" else (0.0, case["t1"],
                                                                               1e-6, 1e-8)
    if case["kind"] == "pleiades":
        return 0.0, 0.1 * case["steps"], 1e-10, 0.0
    return 0.0, 1e-6, RTOL, ATOL


def _host_inputs(case, seed):
    """(y0, g) of a single-problem case as numpy arrays."""
    kind, n = case["kind"], case["n"]
    if kind == "vdp":
        return inputs.vdp_inputs(n, seed, (0.5, 2.0) if case["method"] == "rkck"
                                 else (300.0, 3000.0))
    if kind == "pleiades":
        return inputs.pleiades_inputs(n, seed)
    sp = case["species"]
    if kind == "thermal":
        return inputs.thermal_inputs(_network(sp, True), n, seed, (1000.0, 2500.0))
    return inputs.kinetics_inputs(_network(sp), n, seed, _t_range(sp))


def _problem(case):
    kind = case["kind"]
    if kind == "vdp":
        return rk.Problem.vdp()
    if kind == "pleiades":
        return rk.Problem.pleiades()
    if kind == "thermal":
        return rk.Problem.network_thermal(_network(case["species"], True))
    return rk.Problem.network(_network(case["species"]))


def prepare(case, seed):
    dev = torch.device("cuda:0")
    if case["kind"] == "ragged":
        _, per_net = inputs.ragged_inputs(case["n"], seed, (800.0, 3000.0))
        y0 = [torch.from_numpy(y).to(dev) for y, _ in per_net]
        return dict(case=case, batch=rk.Batch([rk.Problem.network(_network(k))
                                               for k in (9, 13, 32, 53)]),
                    y0=y0, gs=[torch.from_numpy(g).to(dev) for _, g in per_net],
                    ys=[torch.empty_like(y) for y in y0],
                    status=[torch.empty(y.shape[1], dtype=torch.int32, device=dev) for y in y0],
                    stats=[torch.empty((rk.RK_NSTATS, y.shape[1]), dtype=torch.int32, device=dev)
                           for y in y0])
    y0, g = _host_inputs(case, seed)
    state = dict(case=case, prob=_problem(case), y0=torch.from_numpy(y0).to(dev),
                 g=torch.from_numpy(g).to(dev) if g is not None else None)
    if case["kind"] == "solve":
        net = _network(case["species"])
        state["lnA"] = torch.from_numpy(net.lnA.copy()).to(dev).requires_grad_()
        state["y0"].requires_grad_()
        state["w"] = torch.from_numpy(inputs.adjoint_weights(net.n_sp, case["n"], seed)).to(dev)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "ragged":
        for y, y0 in zip(state["ys"], state["y0"]):
            y.copy_(y0)
        state["batch"].integrate_rkc(state["ys"], state["gs"], 0.0, 1e-6, case["substeps"], RTOL,
                                     ATOL, use_graph=case["graph"], status=state["status"],
                                     stats=state["stats"])
        return dict(y=state["ys"], status=state["status"], stats=state["stats"])
    t0, t1, rtol, atol = _interval(case)
    prob, y0, g = state["prob"], state["y0"], state["g"]
    if kind == "solve":
        solve = rk.rkck_solve if case["method"] == "rkck" else rk.rkc_solve
        y1, status, stats = solve(prob, y0, g, t0, t1, rtol, atol, lnA=state["lnA"])
        dy0, dlnA = torch.autograd.grad(y1, (y0, state["lnA"]), state["w"])
        return dict(y1=y1.detach(), status=status, stats=stats, dy0=dy0, dlnA=dlnA)
    step = rk.integrate_rkck if case["method"] == "rkck" else rk.integrate_rkc
    if kind == "pleiades":
        dt = (t1 - t0) / case["steps"]
        y1, stats = y0, []
        for k in range(case["steps"]):
            y1, status, st = step(prob, y1, g, k * dt, (k + 1) * dt, rtol, atol)
            stats.append(st)
        return dict(y1=y1, status=status, stats=stats)
    opts = dict(schedule=case["schedule"])
    if case.get("cost_order"):
        opts["cost_order"] = 1
    y1, status, stats = step(prob, y0, g, t0, t1, rtol, atol, **opts)
    return dict(y1=y1, status=status, stats=stats)


# ------------------------------------------------------------------- work
# Mean right-hand-side evaluations a system's integration takes at these
# tolerances (from the statistics of the standard workloads): what the adaptive
# method needs, not what a kernel spends.
_EVALS = {("vdp", "rkck"): 1310, ("vdp", "rkc"): 2370, ("pleiades", "rkck"): 470,
          (9, "rkc"): 7660, (9, "rkck"): 4530, (13, "rkc"): 2530, (13, "rkck"): 440,
          (32, "rkc"): 12900, (32, "rkck"): 32900, (53, "rkc"): 9900, (53, "rkck"): 16600}


def _per_system(kind, species, method):
    """(bytes in and out, flops) of one system's integration."""
    thermal = kind == "thermal"
    if kind == "vdp":
        n_eq, n_par, per = 2, 1, 5 + 12 * 2
        evals = _EVALS["vdp", method]
    elif kind == "pleiades":
        n_eq, n_par, per = 28, 0, 378 + 10 * 28
        evals = _EVALS["pleiades", method]
    else:
        net = _network(species)
        n_eq, n_par = species + thermal, 1 if thermal else 2
        per = flops.rhs_flops(flops.Thermal(_network(species, True)) if thermal else net)
        per += 10 * n_eq
        evals = _EVALS[species, method]
    return (2 * n_eq + n_par) * 8 + 28, evals * per


def work(case):
    n = case["n"]
    if case["kind"] == "ragged":
        got = [_per_system("net", k, "rkc") for k in (9, 13, 32, 53)]
        # a substep after the first starts past the initial transients
        share = n / 4 * (1.0 + 0.3 * (case["substeps"] - 1))
        return dict(bytes=share * sum(b for b, _ in got), flops=share * sum(f for _, f in got))
    kind = case["kind"]
    b, f = _per_system(kind, case.get("species"), case["method"])
    if kind == "pleiades":
        b *= case["steps"]
    if kind == "solve":
        # the weights in, two gradients out, and a reverse sweep of about twice
        # the forward's operations
        net = _network(case["species"])
        b, f = b + 2 * 8 * net.n_sp, 3 * f
    return dict(bytes=n * b, flops=n * f)


# ------------------------------------------------------------------ exact
# Dormand and Prince's 5(4) pair with a step size per system, far below the
# cases' tolerances.
_A = [[], [1 / 5], [3 / 40, 9 / 40], [44 / 45, -56 / 15, 32 / 9],
      [19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729],
      [9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656],
      [35 / 384, 0.0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84]]
_E = [35 / 384 - 5179 / 57600, 0.0, 500 / 1113 - 7571 / 16695, 125 / 192 - 393 / 640,
      -2187 / 6784 + 92097 / 339200, 11 / 84 - 187 / 2100, -1 / 40]


def _reference(f, y, t1, rtol, atol, h0):
    n = y.shape[1]
    t = torch.zeros(n, dtype=torch.float64, device=y.device)
    h = torch.full_like(t, h0)
    k1 = f(y)
    for _ in range(200000):
        left = t1 - t
        if not bool((left > 0).any()):
            break
        hs = torch.minimum(h, left)
        ks = [k1]
        for row in _A[1:]:
            z = y
            for a, k in zip(row, ks):
                if a:
                    z = z + (a * hs) * k
            ks.append(f(z))
        e = sum(c * k for c, k in zip(_E, ks) if c) * hs
        err = ((e / (atol + rtol * torch.maximum(y.abs(), z.abs()))) ** 2).mean(0).sqrt()
        ok = (err <= 1.0) & (left > 0)
        t = torch.where(ok, torch.where(hs >= left, torch.full_like(t, t1), t + hs), t)
        y = torch.where(ok, z, y)
        k1 = torch.where(ok, ks[-1], k1)
        h = hs * torch.clamp(0.9 * err.clamp_min(1e-30) ** -0.2, 0.2, 5.0)
    return y


def _mass_action(net, T, rho):
    """dY/dt of the isothermal network (T [n] and rho [n] constant)."""
    dev = T.device
    W = torch.as_tensor(net.W, device=dev)[:, None]
    lnA, beta, Ea, K = (torch.as_tensor(a, device=dev)[:, None]
                        for a in (net.lnA, net.beta, net.Ea, net.Keq))
    kf = torch.exp(lnA + beta * torch.log(T) - Ea / T)
    kr = kf / K
    nu = torch.as_tensor(net.stoich(), dtype=torch.float64, device=dev)
    n_sp = net.n_sp
    r, p = (torch.as_tensor(np.where(s < 0, n_sp, s).astype(np.int64), device=dev)
            for s in (net.reac, net.prod))

    def f(Y):
        C = rho * Y / W
        C = torch.cat([C, C.sum(0, keepdim=True)])
        q = kf * C[r[:, 0]] * C[r[:, 1]] - kr * C[p[:, 0]] * C[p[:, 1]]
        return (nu @ q) * W / rho
    return f


def _pleiades(y):
    x, v = y[:14].view(2, 7, -1), y[14:]
    m = torch.arange(1.0, 8.0, dtype=torch.float64, device=y.device)[None, :, None]
    acc = torch.empty_like(x)
    for i in range(7):
        d = x - x[:, i:i + 1]
        r2 = (d * d).sum(0)
        r2[i] = 1.0
        acc[:, i] = (m * d / (r2 * r2.sqrt())).sum(1)
    return torch.cat([v, acc.reshape(14, -1)])


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if kind not in ("vdp", "net", "solve", "pleiades"):
        return None
    if case.get("species", 0) > 13 or (kind == "vdp" and case["method"] == "rkc"):
        return None                    # tens of thousands of explicit steps
    if kind == "pleiades" and n > 20000:
        return None
    dev = torch.device("cuda:0" if torch.cuda.is_available() else "cpu")
    y0, g = (torch.from_numpy(a).to(dev) if a is not None else None
             for a in _host_inputs(case, seed))
    _, t1, _, _ = _interval(case)
    if kind == "vdp":
        mu = g[0]

        def f(y):
            return torch.stack([y[1], mu * (1.0 - y[0] * y[0]) * y[1] - y[0]])
        tol = (1e-11, 1e-13)
    elif kind == "pleiades":
        f, tol = _pleiades, (1e-13, 1e-13)
    else:
        f, tol = _mass_action(_network(case["species"]), g[0], g[1]), (1e-11, 1e-15)
    y1 = _reference(f, y0, t1, *tol, h0=1e-4 * t1)
    if kind == "solve":
        return dict(y1=y1, status=None, stats=None, dy0=None, dlnA=None)
    return dict(y1=y1, status=None, stats=[None] * case["steps"] if kind == "pleiades" else None)
