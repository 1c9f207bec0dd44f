"""Performance cases of the gravity library, over the range its users run it.

A case is a dict of plain values.  ``prepare`` makes what a simulation has in
hand before the call (a context, particle arrays on the GPU, output arrays),
``run`` makes one pass through the public entry points, ``exact`` gives the
same results by direct summation in 64-bit torch where that is affordable,
and ``work`` counts the bytes and operations a pass cannot do without.

Kinds of pass:
  step       every particle: tree build, g/j/T, tidal timestep and bin, due
             list, predictor (the standard scheme's step)
  active     the adaptive scheme's step: a build over all particles and fresh
             forces for a listed subset whose number lies on the device
  direct     direct summation, all or some targets, FP64 or FP32 pair terms
  lengths    adaptive softening: neighbour lengths, rebuild input, softened g
  pm         Price & Monaghan lengths, softened gravity and correction
  periodic   periodic cube, nearest image or Ewald sums
  adjoint    forward and gradient through the autograd function
  batched    many small systems in one build and one evaluation
  integrate  one kick-drift-kick step of the adaptive integrator
"""
from __future__ import annotations

import math

import torch

import paper_2010_13792_amd as ag
from paper_2010_13792_amd.driver import AdaptiveIntegrator

DEV = "cuda:0"
F64 = torch.float64
PP_FLOPS, PN_FLOPS = 57, 179     # a pair and a node interaction as written
DIRECT_FLOPS = 60                # a pair of the direct sum as written
EXACT_PAIRS = 1 << 34            # most pairs of a direct sum that exact() takes
CHUNK_PAIRS = 1 << 24


# ---------------------------------------------------------------------------
# particle sets (total mass 1 per system)
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=F64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=F64)


def _directions(g, n):
    d = _randn(g, n, 3)
    return d / d.norm(dim=1, keepdim=True)


def _plummer_radii(g, n, b=1.0, rmax=10.0):
    s = rmax / b
    mu = s ** 3 / (1.0 + s * s) ** 1.5
    u = (_rand(g, n) * mu).clamp_min(1e-300)
    return b / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)


def _smooth_velocities(g, x, modes=48):
    """A turbulent velocity field: Fourier modes of random direction with
    amplitude falling as k^-2, 3-D rms 1 (the cloud's initial condition)."""
    k = torch.exp(_rand(g, modes) * math.log(16.0)) * math.pi
    kv = _directions(g, modes) * k[:, None]
    amp = _randn(g, modes, 3) * (k ** -2.0)[:, None]
    v = torch.sin(x @ kv.T + 2.0 * math.pi * _rand(g, modes)) @ amp
    v -= v.mean(dim=0)
    return v / v.square().sum(dim=1).mean().sqrt()


def _particles(shape, n, seed):
    """x, v, m of one particle set."""
    g = _gen(seed)
    m = torch.full((n,), 1.0 / n, dtype=F64, device=DEV)
    if shape == "plummer":       # a star cluster: Plummer sphere, scale 1, r <= 10
        x = _directions(g, n) * _plummer_radii(g, n)[:, None]
        v = 0.4 * _randn(g, n, 3)
    elif shape == "sphere":      # a turbulent cloud: uniform unit sphere
        x = _directions(g, n) * (_rand(g, n) ** (1.0 / 3.0))[:, None]
        v = _smooth_velocities(g, x)
    else:                        # "clumps": 64 Plummer clumps in the unit cube
        mc = torch.exp(_randn(g, 64))
        mc /= mc.sum()
        cid = torch.multinomial(mc, n, replacement=True, generator=g).sort().values
        b = 0.02 * (64.0 * mc) ** (1.0 / 3.0)
        r = _plummer_radii(g, n) * b[cid]        # truncated at ten scale lengths
        x = _rand(g, 64, 3)[cid] + _directions(g, n) * r[:, None]
        v = _randn(g, n, 3) * torch.sqrt(math.pi * mc / (32.0 * b))[cid][:, None]
    return x.contiguous(), v.contiguous(), m


def _old_acc(shape, x):
    """The last accelerations the relative opening test compares with."""
    r2 = x.square().sum(dim=1, keepdim=True)
    return (-x / (r2 + 1.0) ** 1.5 if shape == "plummer" else -x).contiguous()


def _pancake(n_side, seed):
    """Periodic unit cube: a lattice displaced by one plane-wave mode."""
    g = _gen(seed)
    q1 = (torch.arange(n_side, device=DEV, dtype=F64) + 0.5) / n_side
    x = torch.stack(torch.meshgrid(q1, q1, q1, indexing="ij"), -1).reshape(-1, 3)
    s = torch.sin(2.0 * math.pi * x[:, 0]) / (2.0 * math.pi)
    x = x.clone()
    x[:, 0] -= 0.9 * s
    x = torch.remainder(x + 1e-3 / n_side * _randn(g, *x.shape), 1.0)
    v = torch.zeros_like(x)
    v[:, 0] = -s
    n = x.shape[0]
    return x.contiguous(), v, torch.full((n,), 1.0 / n, dtype=F64, device=DEV)


def _subset(n, frac, seed):
    g = _gen(seed + 7919)
    k = max(1, round(frac * n))
    return torch.randperm(n, generator=g, device=DEV)[:k].sort().values.to(torch.int32)


def _fields(n):
    z = lambda k: torch.zeros((n, k), dtype=F64, device=DEV)  # noqa: E731
    return {"acc": z(3), "jerk": z(3), "tidal": z(6)}


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest call of a user: one step of a few thousand stars, where latency and launches count
        {"name": "step_plummer_3k", "kind": "step", "shape": "plummer", "n": 3000, "theta": 0.5, "eps": 0.01,
         "alpha": 0.0},
        # the headline workload of bench.py: a cloud of 2^20 particles, every force fresh
        {"name": "step_sphere_1m", "kind": "step", "shape": "sphere", "n": 1 << 20, "theta": 0.7, "eps": 1e-3,
         "alpha": 0.0},
        # the paper code's opening rule (geometric and relative criterion), a ragged number of particles
        {"name": "step_relative_180k", "kind": "step", "shape": "sphere", "n": 180001, "theta": 0.7, "eps": 1e-3,
         "alpha": 0.0025},
        # the method itself at the largest size of bench.py: 2^22 particles in clumps, a tenth due
        {"name": "active_clumps_4m", "kind": "active", "shape": "clumps", "n": 1 << 22, "frac": 0.1, "theta": 0.7,
         "eps": 1e-3},
        # direct summation of a small cluster in double precision
        {"name": "direct_plummer_4096", "kind": "direct", "shape": "plummer", "n": 4096, "frac": 1.0, "eps": 0.01,
         "fp32": False},
        # fully adaptive softening: 32nd-neighbour lengths found on the device every step
        {"name": "lengths_sphere_131k", "kind": "lengths", "shape": "sphere", "n": 1 << 17, "k": 32, "theta": 0.7},
        # the energy-conserving form of adaptive softening
        {"name": "pm_sphere_65k", "kind": "pm", "shape": "sphere", "n": 1 << 16, "n_ngb": 32.0, "theta": 0.7},
        # the paper's cosmological test: 64^3 particles with Ewald sums
        {"name": "periodic_ewald_64", "kind": "periodic", "n_side": 64, "ewald": True, "theta": 0.5},
        # periodic cube with every pair at its nearest image
        {"name": "periodic_near_32", "kind": "periodic", "n_side": 32, "ewald": False, "theta": 0.5},
        # gradients of the forces for inverse problems
        {"name": "adjoint_sphere_100k", "kind": "adjoint", "shape": "sphere", "n": 100003, "theta": 0.6, "eps": 1e-3},
        # an ensemble of small clusters in one call
        {"name": "batched_plummer_64", "kind": "batched", "n_sys": 64, "nmin": 1024, "nmax": 16384, "frac": 0.5,
         "theta": 0.5, "eps": 0.01},
        # the whole engine: one adaptive integrator step
        {"name": "integrate_plummer_32k", "kind": "integrate", "shape": "plummer", "n": 32768, "q_f": 0.25,
         "theta": 0.7, "eps": 0.01, "graph": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "active", "direct", "direct", "lengths", "pm", "periodic", "adjoint",
                       "batched", "integrate"])
    shape = rng.choice(["plummer", "sphere", "clumps"])
    theta = rng.choice([0.5, 0.6, 0.7])
    if kind == "step":
        alpha = 0.0 if shape == "clumps" or rng.random() < 0.6 else rng.choice([0.01, 0.0025])
        n = _log_int(rng, 256, 600000 if alpha == 0.0 else 150000)
        return {"kind": kind, "shape": shape, "n": n, "theta": theta, "eps": rng.choice([1e-3, 0.01]), "alpha": alpha}
    if kind == "active":
        return {"kind": kind, "shape": shape, "n": _log_int(rng, 4096, 2000000),
                "frac": math.exp(rng.uniform(math.log(0.005), math.log(0.6))), "theta": theta, "eps": 1e-3}
    if kind == "direct":
        n = _log_int(rng, 200, 40000)
        return {"kind": kind, "shape": shape, "n": n, "frac": rng.choice([1.0, 1.0, 0.3, 0.05, 0.004]), "eps": 0.01,
                "fp32": rng.random() < 0.5}
    if kind == "lengths":
        return {"kind": kind, "shape": shape, "n": _log_int(rng, 2000, 250000), "k": rng.choice([8, 16, 32, 48, 64]),
                "theta": theta}
    if kind == "pm":
        return {"kind": kind, "shape": shape, "n": _log_int(rng, 2000, 120000), "n_ngb": rng.choice([24.0, 32.0, 40.0]),
                "theta": theta}
    if kind == "periodic":
        ewald = rng.random() < 0.6
        return {"kind": kind, "n_side": rng.randint(9, 60) if ewald else rng.randint(9, 30), "ewald": ewald,
                "theta": theta}
    if kind == "adjoint":
        return {"kind": kind, "shape": shape, "n": _log_int(rng, 500, 100000), "theta": theta, "eps": 1e-3}
    if kind == "batched":
        nmin = rng.choice([200, 512, 1024])
        return {"kind": kind, "n_sys": rng.randint(2, 64), "nmin": nmin, "nmax": nmin * rng.choice([2, 8, 12]),
                "frac": rng.choice([0.1, 0.5, 1.0]), "theta": theta, "eps": 0.01}
    return {"kind": kind, "shape": rng.choice(["plummer", "sphere"]), "n": _log_int(rng, 1500, 100000),
            "q_f": rng.choice([0.0, 0.125, 0.25]), "theta": theta, "eps": 0.01, "graph": rng.random() < 0.4}


def _batch_sizes(case):
    """Sizes spread evenly over the logarithm between nmin and nmax (the
    total number of particles is the case's, not the seed's)."""
    s, lo, hi = case["n_sys"], math.log(case["nmin"]), math.log(case["nmax"])
    return [int(round(math.exp(lo + (hi - lo) * (k + 0.5) / s))) for k in range(s)]


def _soft_guess(x):
    """Lengths of an earlier step: a smooth function of the position."""
    n = x.shape[0]
    return ((0.5 + 0.25 * x.square().sum(dim=1).sqrt()) * 2.0 * n ** (-1.0 / 3.0)).contiguous()


# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "kind": kind}
    if kind == "periodic":
        s["x"], s["v"], s["m"] = _pancake(case["n_side"], seed)
    elif kind == "batched":
        sizes = _batch_sizes(case)
        parts = [_particles("plummer", k, seed * 1009 + i) for i, k in enumerate(sizes)]
        s["x"], s["v"], s["m"] = (torch.cat([p[c] for p in parts]).contiguous() for c in range(3))
        off = [0]
        for k in sizes:
            off.append(off[-1] + k)
        s["off"] = torch.tensor(off, dtype=torch.int64, device=DEV)
        s["idx"] = _subset(off[-1], case["frac"], seed)
    else:
        s["x"], s["v"], s["m"] = _particles(case["shape"], case["n"], seed)
    n = s["x"].shape[0]
    stream = torch.cuda.Stream() if case.get("graph") else None
    if stream is not None:
        stream.wait_stream(torch.cuda.current_stream())
    s["ctx"] = c = ag.Context(0, stream)
    if kind == "integrate":
        s["integ"] = AdaptiveIntegrator(c, s["x"], s["v"], s["m"], q_f=case["q_f"], theta=case["theta"],
                                        eps=case["eps"], step_shift=2)
        if case["graph"]:
            s["integ"].capture()
        return s
    s.update(_fields(n))
    if kind in ("step", "active"):
        s["dt"] = torch.zeros(n, dtype=F64, device=DEV)
        s["bins"] = torch.zeros(n, dtype=torch.int8, device=DEV)
        s["pred"] = torch.zeros((n, 3), dtype=F64, device=DEV)
        s["age"] = torch.zeros(n, dtype=torch.int64, device=DEV)
    if kind == "step":
        s["due"] = torch.zeros(n, dtype=torch.int32, device=DEV)
        s["n_due"] = torch.zeros(1, dtype=torch.int64, device=DEV)
        s["t0"] = torch.zeros(n, dtype=F64, device=DEV)
        if case["alpha"] > 0.0:
            s["old"] = _old_acc(case["shape"], s["x"])
    elif kind == "active":
        idx = _subset(n, case["frac"], seed)
        s["k"] = idx.shape[0]
        s["idx"] = torch.zeros(n, dtype=torch.int32, device=DEV)
        s["idx"][:s["k"]] = idx
        s["n_idx"] = torch.full((1,), s["k"], dtype=torch.int64, device=DEV)
        s["total"] = torch.zeros(1, dtype=torch.int64, device=DEV)
        s["age"] += 1
        s["age"][idx.long()] = 0
    elif kind == "direct":
        s["idx"] = None if case["frac"] >= 1.0 else _subset(n, case["frac"], seed)
    elif kind == "lengths":
        s["h"] = _soft_guess(s["x"])
        c.set_softening(s["h"])
        s["h_new"] = torch.zeros(n, dtype=F64, device=DEV)
    elif kind == "pm":
        s["h"], s["omega"], s["z"] = (torch.zeros(n, dtype=F64, device=DEV) for _ in range(3))
        s["corr"] = torch.zeros((n, 3), dtype=F64, device=DEV)
    elif kind == "periodic":
        c.set_periodic(1.0, case["ewald"])
    elif kind == "adjoint":
        s["x"].requires_grad_(True)
        s["m"].requires_grad_(True)
        s["w"] = _randn(_gen(seed + 31337), n, 3)
    return s


def run(s):
    case, kind, c = s["case"], s["kind"], s["ctx"]
    x, v, m = s["x"], s["v"], s["m"]
    if kind == "integrate":
        it = s["integ"]
        it.step()
        return {"x": it.x, "v": it.v, "acc": it.acc, "tidal": it.tidal, "bins": it.bins, "age": it.tf}
    if kind == "adjoint":
        acc, jerk, tidal = ag.grav_eval(c, x, v, m, None, case["theta"], case["eps"])
        dx, dm = torch.autograd.grad(acc, (x, m), s["w"])
        return {"acc": acc, "jerk": jerk, "tidal": tidal, "dx": dx, "dm": dm}
    acc, jerk, tidal = s["acc"], s["jerk"], s["tidal"]
    out = {"acc": acc, "jerk": jerk, "tidal": tidal}
    if kind == "step":
        c.tree_build(x, v, m, 16)
        if case["alpha"] > 0.0:
            c.set_relative_opening(case["alpha"], s["old"])
        c.grav_eval(None, case["theta"], case["eps"], 1.0, acc, jerk, tidal)
        c.grav_timestep(tidal, 0.01, 1.0, 30, s["dt"], s["bins"])
        c.adaptive_select(s["age"], s["bins"], 1, 16, 0.125, s["due"], s["n_due"], t0=s["t0"], t=1.0)
        c.grav_predict(acc, jerk, s["t0"], 1.0 + 1e-4, s["pred"])
        return {**out, "dt": s["dt"], "bins": s["bins"], "age": s["age"], "n_due": s["n_due"], "pred": s["pred"]}
    if kind == "active":
        c.tree_build(x, v, m, 16)
        c.grav_eval_dev(s["idx"], s["n_idx"], case["theta"], case["eps"], 1.0, acc, jerk, tidal, n_total=s["total"])
        c.grav_timestep_dev(tidal, 0.01, 1.0, 30, s["dt"], s["bins"], s["idx"], s["n_idx"])
        c.grav_predict_age(acc, jerk, s["age"], 1e-4, s["pred"])
        return {**out, "dt": s["dt"], "bins": s["bins"], "pred": s["pred"], "total": s["total"]}
    if kind == "direct":
        c.grav_direct(x, v, m, s["idx"], case["eps"], 1.0, acc, jerk, tidal,
                      precision=ag.AG_FP32_PAIRS if case["fp32"] else ag.AG_FP64)
        return out
    if kind == "lengths":   # softened with the lengths of the step before; new ones for the next
        c.tree_build(x, v, m, 16)
        c.grav_eval(None, case["theta"], 1e-3, 1.0, acc, jerk, tidal)
        c.neighbour_lengths(case["k"], s["h_new"])
        c.set_softening(s["h_new"])
        return {**out, "h": s["h_new"]}
    if kind == "pm":
        c.set_softening()
        c.tree_build(x, v, m, 16)
        c.pm_lengths(case["n_ngb"], s["h"], s["omega"])
        c.set_softening(s["h"])
        c.tree_build(x, v, m, 16)
        c.grav_eval(None, case["theta"], 1e-3, 1.0, acc, jerk, tidal)
        c.pm_factors(case["n_ngb"], 1.0, s["omega"], s["z"])
        c.pm_correct(s["z"], s["corr"])
        return {**out, "h": s["h"], "omega": s["omega"], "z": s["z"], "corr": s["corr"]}
    if kind == "periodic":
        c.tree_build(x, v, m, 16)
        c.grav_eval(None, case["theta"], 0.125 / case["n_side"], 1.0, acc, jerk, tidal)
        return out
    c.tree_build_batched(x, v, m, s["off"], 16)
    c.grav_eval_batched(s["idx"], case["theta"], case["eps"], 1.0, acc, jerk, tidal)
    return out


# ---------------------------------------------------------------------------
def _count(case):
    """(particles, targets)"""
    if case["kind"] == "periodic":
        return case["n_side"] ** 3, case["n_side"] ** 3
    if case["kind"] == "batched":
        n = sum(_batch_sizes(case))
    else:
        n = case["n"]
    return n, max(1, round(case.get("frac", 1.0) * n))


def _tree_flops(n, k, theta):
    """Targets times a tree walk's interactions: near 550 of each sort at
    theta = 0.7 and 2^20 particles, growing with log n and as theta^-2."""
    per = min(n, 27.0 * math.log2(max(n, 2)) * (0.7 / theta) ** 2)
    return k * per * (PP_FLOPS + PN_FLOPS)


def work(case):
    kind = case["kind"]
    n, k = _count(case)
    build = 56.0 * n                  # x, v, m once
    fields = 96.0 * k                 # g, j, T of every target once
    if kind == "direct":
        return {"bytes": 56.0 * n + fields, "flops": float(DIRECT_FLOPS) * n * k}
    flops = _tree_flops(n, k, case["theta"])
    if kind == "step":
        # dt, bin, due list, counters, t0 and the prediction
        return {"bytes": build + fields + n * (9 + 4 + 16 + 8 + 24.0) + (24.0 * n if case["alpha"] > 0.0 else 0.0),
                "flops": flops}
    if kind == "active":
        return {"bytes": build + fields + 4.0 * k + 9.0 * k + n * (48 + 8 + 24.0), "flops": flops}
    if kind == "lengths":             # distances to k neighbours, at eight operations each
        return {"bytes": build + fields + 16.0 * n, "flops": flops + 8.0 * n * case["k"]}
    if kind == "pm":                  # a solve, the factors and the correction over the pairs of each support
        return {"bytes": build + fields + 48.0 * n, "flops": flops + n * case["n_ngb"] * (5 * 20 + 25 + 45.0)}
    if kind == "adjoint":             # the walk for the fields, then one for the gradient
        return {"bytes": build + fields + 56.0 * n, "flops": 2.0 * flops}
    if kind == "integrate":           # positions, velocities, forces and jerks through the predictor and both kicks
        return {"bytes": build + 240.0 * n, "flops": flops * (1.0 if case["q_f"] == 0.0 else 0.5)}
    return {"bytes": build + fields, "flops": flops}


# ---------------------------------------------------------------------------
# the same quantities by direct summation in 64 bits
# ---------------------------------------------------------------------------
def _spline(r2, h):
    """Force factor f and D = f'/r of a unit mass spread by the cubic spline
    of support h (Newtonian beyond it)."""
    r = r2.sqrt()
    u = r / h
    rs = torch.where(r2 > 0, r2, 1.0)
    fn = rs ** -1.5
    inner, soft = u < 0.5, u < 1.0
    us = u.clamp_min(0.5)
    f1 = (32.0 / 3.0 + u * u * (-38.4 + 32.0 * u)) / h ** 3
    d1 = (96.0 * u - 76.8) / h ** 5
    f2 = (64.0 / 3.0 - 48.0 * us + 38.4 * us ** 2 - 32.0 / 3.0 * us ** 3 - 1.0 / (15.0 * us ** 3)) / h ** 3
    d2 = (-48.0 / us + 76.8 - 32.0 * us + 0.2 / us ** 5) / h ** 5
    f = torch.where(inner, f1, torch.where(soft, f2, fn))
    d = torch.where(inner, d1, torch.where(soft, d2, -3.0 * fn / rs))
    return f, d


def _erf_part(r2, alpha):
    """Long-range complement B - 1/r^3 of an Ewald split and its C = B'/r."""
    r = r2.sqrt()
    z = (alpha * r).clamp_min(0.05)
    r = z / alpha
    e = 2.0 / math.sqrt(math.pi) * alpha * torch.exp(-z * z)
    b = -(torch.erf(z) / r ** 3 - e / r ** 2)
    c = -(-3.0 * torch.erf(z) / r ** 5 + e * (3.0 / r ** 4 + 2.0 * alpha ** 2 / r ** 2))
    near = alpha * r2.sqrt() < 0.3      # series of the same: the closed form cancels there
    z2 = alpha ** 2 * r2
    p = 2.0 / math.sqrt(math.pi)
    bs, cs, fact = torch.zeros_like(r2), torch.zeros_like(r2), 1.0
    for k in range(1, 12):
        fact *= k
        a = (-1.0) ** k * 2.0 * k / ((2.0 * k + 1.0) * fact) * p
        bs = bs + a * alpha ** 3 * z2 ** (k - 1)
        if k > 1:
            cs = cs + a * (2.0 * k - 2.0) * alpha ** 5 * z2 ** (k - 2)
    return torch.where(near, bs, b), torch.where(near, cs, c)


def _direct64(x, v, m, rows, h, box=0.0, ewald=False):
    """acc, jerk, tidal at the rows (all: None); h a length or one per particle."""
    n = x.shape[0]
    rows = torch.arange(n, device=DEV) if rows is None else rows.long()
    acc, jerk, tid = (torch.zeros((n, k), dtype=F64, device=DEV) for k in (3, 3, 6))
    step = max(1, CHUNK_PAIRS // n)
    per = torch.is_tensor(h)
    alpha = 4.0 / box if ewald else 0.0
    shifts = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)] if ewald else []
    for r0 in range(0, rows.shape[0], step):
        i = rows[r0:r0 + step]
        d = [x[None, :, a] - x[i, None, a] for a in range(3)]
        if box > 0.0:
            d = [q - box * torch.round(q / box) for q in d]
        nu = [v[None, :, a] - v[i, None, a] for a in range(3)]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        if per:
            f1, d1 = _spline(r2, h[i, None])
            f2, d2 = _spline(r2, h[None, :])
            f, D = 0.5 * (f1 + f2), 0.5 * (d1 + d2)
        else:
            f, D = _spline(r2, torch.as_tensor(h, dtype=F64, device=DEV))
        f = f * m[None]
        D = D * m[None]
        at = torch.arange(i.shape[0], device=DEV)
        f[at, i] = 0.0
        D[at, i] = 0.0
        s = D * (d[0] * nu[0] + d[1] * nu[1] + d[2] * nu[2])
        for a in range(3):
            jerk[i, a] = (f * nu[a] + s * d[a]).sum(1)
        parts = [(f, D, d)]
        for sh in shifts:
            y = [d[a] + box * sh[a] for a in range(3)]
            q2 = y[0] * y[0] + y[1] * y[1] + y[2] * y[2]
            b, c = _erf_part(q2, alpha)
            if sh != (0, 0, 0):
                b, c = b + q2 ** -1.5, c - 3.0 * q2 ** -2.5
            parts.append((b * m[None], c * m[None], y))
        for b, c, y in parts:
            for a in range(3):
                acc[i, a] += (b * y[a]).sum(1)
                tid[i, a] -= (b + c * y[a] * y[a]).sum(1)
            for q, (a, e) in enumerate(((0, 1), (0, 2), (1, 2))):
                tid[i, 3 + q] -= (c * y[a] * y[e]).sum(1)
    if ewald:   # the reciprocal sum, by structure factors
        kf = 2.0 * math.pi / box
        hh = torch.arange(-8, 9, device=DEV, dtype=F64)
        kv = kf * torch.stack(torch.meshgrid(hh, hh, hh, indexing="ij"), -1).reshape(-1, 3)
        k2 = kv.square().sum(1)
        keep = (k2 > 0) & (k2 < 65.0 * kf * kf)
        kv, k2 = kv[keep], k2[keep]
        w = 4.0 * math.pi / box ** 3 * torch.exp(-k2 / (4.0 * alpha ** 2)) / k2
        for q in range(0, kv.shape[0], 256):
            kq, wq = kv[q:q + 256], w[q:q + 256]
            ph = x @ kq.T
            cs, sn = torch.cos(ph), torch.sin(ph)
            C, S = m @ cs, m @ sn
            sin_d = cs * S - sn * C          # sum_j m_j sin(k.(x_j - x_i))
            cos_d = cs * C + sn * S
            acc += (sin_d * wq) @ kq
            kk = torch.stack([kq[:, a] * kq[:, b] for a, b in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))], 1)
            tid -= (cos_d * wq) @ kk
    return acc, jerk, tid


def _adjoint64(x, m, w, eps):
    """Gradient of sum_k w_k . g_k with respect to x and m."""
    n = x.shape[0]
    dx, dm = torch.zeros((n, 3), dtype=F64, device=DEV), torch.zeros(n, dtype=F64, device=DEV)
    step = max(1, CHUNK_PAIRS // n)
    for r0 in range(0, n, step):
        i = torch.arange(r0, min(n, r0 + step), device=DEV)
        d = [x[None, :, a] - x[i, None, a] for a in range(3)]
        f, D = _spline(d[0] * d[0] + d[1] * d[1] + d[2] * d[2], torch.as_tensor(eps, dtype=F64, device=DEV))
        at = i - r0
        f[at, i] = 0.0
        D[at, i] = 0.0
        # d(w_i . g_i) / dx_i = -sum_j m_j J w_i; d(w_j . g_j) / dx_i = m_i J w_j
        q = [m[i, None] * w[None, :, a] - m[None, :] * w[i, None, a] for a in range(3)]
        dq = D * (d[0] * q[0] + d[1] * q[1] + d[2] * q[2])
        for a in range(3):
            dx[i, a] = (f * q[a] + dq * d[a]).sum(1)
        dm[i] = -(f * (d[0] * w[None, :, 0] + d[1] * w[None, :, 1] + d[2] * w[None, :, 2])).sum(1)
    return dx, dm


def _d2(x, i):
    d = x[None] - x[i, None]
    return (d[..., 0] ** 2 + d[..., 1] ** 2) + d[..., 2] ** 2


def _m4(u):
    w = torch.where(u < 0.5, 1.0 + u * u * (6.0 * u - 6.0), 2.0 * (1.0 - u).clamp_min(0.0) ** 3)
    wp = torch.where(u < 0.5, u * (18.0 * u - 12.0), -6.0 * (1.0 - u).clamp_min(0.0) ** 2)
    return w, wp


def _pm64(x, m, n_ngb):
    """Price & Monaghan lengths, Omega, factors and correction."""
    n = x.shape[0]
    near = min(n - 1, 320)
    h, om, z = (torch.zeros(n, dtype=F64, device=DEV) for _ in range(3))
    corr = torch.zeros((n, 3), dtype=F64, device=DEV)
    step = max(1, CHUNK_PAIRS // n)
    target = 3.0 * n_ngb / 32.0
    for r0 in range(0, n, step):
        i = torch.arange(r0, min(n, r0 + step), device=DEV)
        q2 = _d2(x, i)
        q2[i - r0, i] = math.inf
        q2, j = q2.topk(near, largest=False)
        r = q2.sqrt()
        lo, hi = torch.zeros_like(r[:, 0]), r[:, -1].clone()
        for _ in range(70):
            mid = 0.5 * (lo + hi)
            s = 1.0 + _m4(r / mid[:, None])[0].sum(1)
            lo, hi = torch.where(s < target, mid, lo), torch.where(s < target, hi, mid)
        hh = 0.5 * (lo + hi)
        u = r / hh[:, None]
        om[i] = -32.0 / (9.0 * n_ngb) * (u * _m4(u)[1]).sum(1)
        h[i] = hh
        # -h^2 dphi/dh of the spread unit mass: psi + u psi'
        a = 16.0 * u ** 2 - 48.0 * u ** 4 + 38.4 * u ** 5 - 2.8
        b = 32.0 * u ** 2 - 64.0 * u ** 3 + 48.0 * u ** 4 - 12.8 * u ** 5 - 3.2
        dphi = -torch.where(u < 0.5, a, torch.where(u < 1.0, b, 0.0))
        dens = 3.0 * n_ngb / (4.0 * math.pi * hh ** 3)
        z[i] = 0.5 * m[i] * hh / (3.0 * dens * om[i]) * (m[j] * dphi).sum(1) / hh ** 2
    for r0 in range(0, n, step):
        i = torch.arange(r0, min(n, r0 + step), device=DEV)
        r = _d2(x, i).sqrt()
        k = 8.0 / math.pi
        c = z[i, None] * k / h[i, None] ** 4 * _m4(r / h[i, None])[1] + z[None] * k / h[None] ** 4 * _m4(r / h[None])[1]
        c = torch.where(r > 0, c / r, 0.0)
        for a in range(3):
            corr[i, a] = -(c * (x[None, :, a] - x[i, None, a])).sum(1) / m[i]
    return h, om, z, corr


def exact(case, seed):
    """What run() returns on its first pass, by direct summation (tree walks
    approximate it); None for what has no such value or would take too long
    (counters and bins follow from the walk's own tidal tensor)."""
    kind = case["kind"]
    n, k = _count(case)
    if kind == "integrate":
        return None
    if kind == "batched":
        sizes = _batch_sizes(case)
        if sum(q * q for q in sizes) > EXACT_PAIRS:
            return None
        idx = _subset(n, case["frac"], seed)
        parts, r0 = [], 0
        for s_i, q in enumerate(sizes):
            x, v, m = _particles("plummer", q, seed * 1009 + s_i)
            rows = idx[(idx >= r0) & (idx < r0 + q)] - r0
            parts.append(_direct64(x, v, m, rows, case["eps"]))
            r0 += q
        acc, jerk, tidal = (torch.cat([p[c] for p in parts]) for c in range(3))
        return {"acc": acc, "jerk": jerk, "tidal": tidal}
    if kind == "periodic":
        if n * n * (27 if case["ewald"] else 1) > EXACT_PAIRS:
            return None
        x, v, m = _pancake(case["n_side"], seed)
        acc, jerk, tidal = _direct64(x, v, m, None, 0.125 / case["n_side"], 1.0, case["ewald"])
        return {"acc": acc, "jerk": jerk, "tidal": tidal}
    if n * k > EXACT_PAIRS or (kind == "pm" and n * n > EXACT_PAIRS // 4):
        return None
    x, v, m = _particles(case["shape"], n, seed)
    if kind == "adjoint":
        w = _randn(_gen(seed + 31337), n, 3)
        acc, jerk, tidal = _direct64(x, v, m, None, case["eps"])
        dx, dm = _adjoint64(x, m, w, case["eps"])
        return {"acc": acc, "jerk": jerk, "tidal": tidal, "dx": dx, "dm": dm}
    if kind == "lengths":
        h = torch.zeros(n, dtype=F64, device=DEV)
        if n * n <= EXACT_PAIRS // 4:
            step = max(1, CHUNK_PAIRS // n)
            for r0 in range(0, n, step):
                i = torch.arange(r0, min(n, r0 + step), device=DEV)
                q = _d2(x, i)
                q[i - r0, i] = math.inf
                h[i] = q.topk(case["k"], largest=False).values[:, -1].sqrt()
        else:
            h = None
        acc, jerk, tidal = _direct64(x, v, m, None, _soft_guess(x))
        return {"acc": acc, "jerk": jerk, "tidal": tidal, "h": h}
    if kind == "pm":
        h, om, z, corr = _pm64(x, m, case["n_ngb"])
        acc, jerk, tidal = _direct64(x, v, m, None, h)
        return {"acc": acc, "jerk": jerk, "tidal": tidal, "h": h, "omega": om, "z": z, "corr": corr}
    rows = None
    if kind == "active" or (kind == "direct" and case["frac"] < 1.0):
        rows = _subset(n, case["frac"], seed)
    acc, jerk, tidal = _direct64(x, v, m, rows, case["eps"])
    out = {"acc": acc, "jerk": jerk, "tidal": tidal}
    if kind == "direct":
        return out
    if kind == "step":     # every row is due or not by its bin: the prediction of a row that is not starts at t0 = 0
        return {**out, "dt": None, "bins": None, "age": None, "n_due": None, "pred": None}
    age = torch.ones(n, dtype=F64, device=DEV)
    age[rows.long()] = 0.0
    return {**out, "dt": None, "bins": None, "pred": acc + jerk * (age * 1e-4)[:, None], "total": None}
