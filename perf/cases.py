"""The work whose speed is measured: whole uncertainty-quantification jobs and
the other calls a program makes, from the smallest to the largest.

A pass is what a user's program does for one answer: it creates a job from a
problem, advances it, and reads the statistics. Two passes differ from that:
a program that watches a running job (a kept job, a few steps and a scalar
statistic per pass) and a program that feeds a server.

Sizes are those of the package's own workloads (the vortex on 64^2, 128^2
and 256^2 lattices, the 440 x 82 cylinder channel, the paper's cylinder, the
four-dimensional vortex study, the serving mix) with fewer time steps per
pass, and generic odd ones. Problems whose class a program runs again and
again have their launch shape tuned once beforehand, as the benchmark and the
studies do; the others run as they come.

The seed moves the input ranges by some per cent and seeds the Monte Carlo
and Latin hypercube draws.
"""
import math
import random

import numpy as np
import torch

import paper_2508_13867_amd as U
from paper_2508_13867_amd import workloads as W

STORED_BYTES = {"fp64": 8, "fp32": 4, "fp16s": 2, "bf16s": 2}
FLOPS_PER_UPDATE = 76  # of one node's collision, a fused multiply-add counted as two


# ------------------------------------------------------------------ cases
def listed():
    return [
        # a program that watches a small job: 16 steps, then the energy's
        # statistics, again and again: launches and host time count
        dict(name="watch96_fp32", kind="watch", nx=96, ny=96, precision="fp32", dims=2, rule="gl", n=3, order=2,
             steps=16, qois="ke"),
        # the smallest whole job: uncertain viscosity at 5 collocation nodes
        dict(name="vortex64_fp64_gl5", kind="vortex", nx=64, ny=64, precision="fp64", dims=1, rule="gl", n=5, order=4,
             steps=1000, qois="ke"),
        # one pair of resolutions of the convergence study in W_1
        dict(name="law4d_fp64_32_64", kind="law", n=32, n2=64, precision="fp64", steps=2000),
        # sparse-grid collocation of the vortex with four inputs
        dict(name="vortex128_smolyak", kind="vortex", nx=128, ny=128, precision="fp32", dims=4, rule="smolyak", n=3,
             order=3, steps=1000, qois="ke,speed"),
        # the benchmark's job
        dict(name="vortex256_gl4x4", kind="vortex", nx=256, ny=256, precision="fp32", dims=4, rule="gl", n=4, order=3,
             steps=2000, qois="ke,vel", tune=True),
        # the Monte Carlo sweep in 16-bit storage, with field statistics
        dict(name="vortex128_mc4096_fp16s", kind="vortex", nx=128, ny=128, precision="fp16s", dims=4, rule="mc",
             n=4096, order=0, steps=400, qois="ke,vel", tune=True),
        # few samples on a large lattice
        dict(name="vortex1024_gl16", kind="vortex", nx=1024, ny=1024, precision="fp32", dims=2, rule="gl", n=4,
             order=3, steps=240, qois="ke"),
        # an odd lattice in double precision with quasi Monte Carlo points
        dict(name="vortex300x190_fp64", kind="vortex", nx=300, ny=190, precision="fp64", dims=2, rule="halton", n=100,
             order=0, steps=333, qois="ke,vel", tune=True),
        # the cylinder channel: drag and lift
        dict(name="channel440x82_gl8x8", kind="channel", nx=440, ny=82, precision="fp32", D=20, dims=2, rule="gl", n=8,
             order=7, steps=3000, qois="cd,cl", tune=True),
        # the serving mix's widest channel
        dict(name="channel880x164_gl32", kind="channel", nx=880, ny=164, precision="fp32", D=40, dims=1, rule="gl",
             n=32, order=3, steps=500, qois="cd"),
        # the paper's own cylinder set-up: curved wall, interpolated ends
        dict(name="paper440x80_gl11", kind="paper", nx=440, ny=80, precision="fp32", D=20, dims=1, rule="gl", n=11,
             order=10, steps=2000, qois="cd,vel"),
        # a server that is handed a mix of jobs at once
        dict(name="serve12", kind="serve", jobs=12, mix=7, precision="fp32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["watch", "vortex", "vortex", "vortex", "channel", "channel", "paper", "law", "serve"])
    if kind == "serve":
        return dict(kind="serve", jobs=rng.randint(4, 12), mix=rng.randint(100, 999), precision="fp32")
    if kind == "law":
        n = rng.choice([8, 12, 16, 24, 32])
        return dict(kind="law", n=n, n2=2 * n, precision=rng.choice(["fp64", "fp32"]), steps=_log(rng, 200, 2000))
    case = dict(kind=kind, precision=rng.choice(["fp32", "fp32", "fp32", "fp64", "fp16s", "bf16s"]))
    if kind in ("watch", "vortex"):
        hi = 160 if kind == "watch" else 1024
        nx = _log(rng, 48, hi)
        ny = nx if rng.random() < 0.5 else min(hi, max(32, int(nx * rng.uniform(0.5, 1.5))))
        if rng.random() < 0.5:  # as often round as odd
            nx, ny = max(32, nx // 32 * 32), max(32, ny // 32 * 32)
        case.update(nx=nx, ny=ny, qois="ke")
        rules = ["gl", "mc", "halton", "lhs", "smolyak"]
        dims = rng.randint(1, 4)
        qois = ["ke"] if dims == 1 else ["ke", "ke,vel", "ke,speed", "ke,rho"]
        if case["precision"] in ("fp16s", "bf16s"):  # inputs that 16 bits resolve
            dims, qois = 4, ["ke", "ke,vel"]
    else:
        D = rng.randint(10, 40)
        case.update(nx=22 * D, ny=4 * D if kind == "paper" else int(round(4.1 * D)), D=D)
        rules = ["gl", "gl", "mc", "halton"]
        qois = ["cd", "cd,vel"]
        dims = 1 if kind == "paper" else rng.randint(1, 2)
    rule = rng.choice(rules)
    if rule == "gl":
        n = rng.randint(2, {1: 16, 2: 12, 3: 5, 4: 4}[dims])
        S, order = n ** dims, min(n - 1, 3)
    elif rule == "smolyak":
        n, order = rng.randint(1, 3), 2
        S = {1: 5, 2: 21, 3: 50, 4: 100}[dims]
    else:
        n = S = _log(rng, 8, 1024)
        order = 0
    cells = case["nx"] * case["ny"]
    while S * cells > 1.2e7 and rule not in ("gl", "smolyak"):
        n = S = n // 2
    while S * cells > 1.2e7 and rule == "gl" and n > 2:
        n -= 1
        S, order = n ** dims, min(n - 1, 3)
    case.update(dims=dims, rule=rule, n=n, order=order)
    if kind == "watch":
        case.update(steps=rng.randint(2, 64))
    else:
        case.update(steps=max(20, min(_log(rng, 100, 3000), int(2.0e9 / (S * cells)))), qois=rng.choice(qois))
        if kind != "paper" and rng.random() < 0.3:
            case["tune"] = True
    return case


# ------------------------------------------------------------------ problems
def _problem(case, seed):
    """The problem of a case; the seed moves its ranges."""
    rng = random.Random(seed)
    nudge = lambda: 1.0 + 0.05 * rng.uniform(-1.0, 1.0)  # noqa: E731
    rule = dict(kind=case["rule"])
    if case["rule"] == "gl":
        rule.update(n=case["n"], order=case["order"])
    elif case["rule"] == "smolyak":
        rule.update(level=case["n"], order=case["order"])
    else:
        rule.update(N=case["n"], seed=seed)
    nx, ny, prec = case["nx"], case["ny"], case["precision"]
    if case["kind"] in ("watch", "vortex"):
        a, b = nudge(), nudge()
        dists = [("nu", 0.004 * a, 0.006 * a), ("u0", 0.018 * b, 0.022 * b), ("phase_x", 0.0, 2 * math.pi),
                 ("phase_y", 0.0, 2 * math.pi)][:case["dims"]]
        return dict(geometry="tgv", precision=prec, nx=nx, ny=ny, u0=0.02, nu=0.005, dists=dists, rule=rule)
    D = case["D"]
    if case["kind"] == "channel":
        a, b = nudge(), nudge()
        dists = [("re", 16.0 * a, 24.0 * a), ("u_peak", 0.045 * b, 0.055 * b)][:case["dims"]]
        return dict(geometry="channel", precision=prec, nx=nx, ny=ny, u_peak=0.05, nu=0.05 * D / 20.0, D=D, cx=2 * D,
                    cy=ny // 2, ramp=case["steps"] // 5, xbc="zouhe", dists=dists, rule=rule)
    a = nudge()
    return dict(geometry="channel", precision=prec, nx=nx, ny=ny, u_peak=0.06, nu=0.04 * D / 20.0, cyl_bc="bouzidi",
                cyl_x=2.0 * D, cyl_y=0.5 * (ny - 1), cyl_d=float(D), ramp=case["steps"] // 5, xbc="interp",
                force_ref="mean", layout="ab", dists=[("u_peak", 0.048 * a, 0.072 * a)], rule=rule)


def _law(case, seed, n):
    """The perturbed vortex at resolution n, and its lattice velocity."""
    a = 1.0 + 0.05 * random.Random(seed).uniform(-1.0, 1.0)
    Ma, Re = 1.6 / n, 40.0 * n * a
    u = Ma / math.sqrt(3.0)
    dx = 2.0 * math.pi / (n - 1)
    return W.tgv4d(n, dict(nu=dx * u / (Re * dx * dx), u_lat=u), precision=case["precision"], seed=seed), u


def _mix(case, seed):
    """The serving mix's jobs: sizes by the case, draws by the seed."""
    trace = W.serving_trace(n_jobs=case["jobs"], seed=case["mix"], max_S_steps=2.4e4, steps_range=(200, 1000))
    jobs = []
    for k, (_, spec) in enumerate(trace):
        spec = dict(spec, dists=[(t, lo * (1 + 1e-3 * (seed % 97)), hi * (1 + 1e-3 * (seed % 97)))
                                 for t, lo, hi in spec["dists"]])
        if spec["rule"]["kind"] == "mc":
            spec["rule"] = dict(spec["rule"], seed=seed + k)
        jobs.append(spec)
    return jobs


# ------------------------------------------------------------------ passes
def _table(results):
    """The jobs' answers side by side, coefficients one after the other."""
    out = {k: np.array([r[k] for r in results]) for k in ("S", "K", "mean", "var", "var_alt")}
    return dict(out, coeffs=np.concatenate([r["coeffs"] for r in results]))


_tuned = set()  # problem classes whose launch shape this process has tuned


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        return dict(kind=kind, server=U.Server(memory_budget_gb=16.0, max_jobs=64, steps_per_tick=96,
                                               precision=case["precision"]), jobs=_mix(case, seed))
    if kind == "law":
        return dict(kind=kind, pair=[_law(case, seed + k, case[n]) for k, n in enumerate(("n", "n2"))],
                    steps=case["steps"])
    spec = _problem(case, seed)
    if case.get("tune"):
        key = (spec["geometry"], case["precision"], case["nx"], case["ny"], case["rule"], case["n"], case["dims"])
        if key not in _tuned:
            U.autotune(spec, steps=20)
            _tuned.add(key)
    state = dict(kind=kind, spec=spec, steps=case["steps"], qois=case["qois"].split(","))
    if kind == "watch":
        state["job"] = U.Job(spec)
    return state


def run(state):
    kind = state["kind"]
    if kind == "watch":
        state["job"].run(state["steps"])
        return {q: state["job"].moments(q) for q in state["qois"]}
    if kind == "serve":
        server = state["server"]
        tickets = [server.submit(spec) for spec in state["jobs"]]
        return _table([server.wait(t) for t in tickets])
    if kind == "law":
        (sa, ua), (sb, ub) = state["pair"]
        with U.Job(sa) as a, U.Job(sb) as b:
            a.run(state["steps"])
            b.run(state["steps"])
            return {"w1": U.wasserstein1(a, b, "speed", 1.0 / ua, 1.0 / ub)}
    with U.Job(state["spec"]) as job:
        job.run(state["steps"])
        return {q: job.moments(q) for q in state["qois"]}


def _samples(spec):
    r = spec["rule"]
    d = len(spec["dists"])
    if r["kind"] == "gl":
        return r["n"] ** d
    if r["kind"] == "smolyak":
        return len(_smolyak(d, r["level"])[1])
    return r["N"]


def work(case):
    """The populations written at the start and read at the end, the
    statistics written, and the collisions."""
    if case["kind"] == "serve":
        jobs = [(s, s["steps"], 1) for s in _mix(case, 0)]
    elif case["kind"] == "law":
        jobs = [(_law(case, 0, case[n])[0], case["steps"], 0) for n in ("n", "n2")]
    else:
        spec = _problem(case, 0)
        cells = spec["nx"] * spec["ny"]
        terms = 3 + len(_multi_indices(case["dims"], case["order"])) * (case["rule"] in ("gl", "smolyak"))
        outs = sum({"vel": 2 * cells, "speed": cells, "rho": cells}.get(q, 1) for q in case["qois"].split(","))
        jobs = [(spec, case["steps"], outs * terms)]
    total, flops = 0.0, 0.0
    for spec, steps, outs in jobs:
        nodes = float(_samples(spec)) * spec["nx"] * spec["ny"]
        total += 18.0 * STORED_BYTES[spec["precision"]] * nodes + 8.0 * outs
        flops += FLOPS_PER_UPDATE * nodes * steps
    return {"bytes": total, "flops": flops}


# ------------------------------------------------------------------ the same in 64 bits
CX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
CY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)
WT = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4


def _multi_indices(d, P):
    if d == 1:
        return [(k,) for k in range(P + 1)]
    every = []

    def go(prefix, left):
        if len(prefix) == d - 1:
            every.append((*prefix, left))
        else:
            for v in range(left, -1, -1):
                go((*prefix, v), left - v)

    for g in range(P + 1):
        go((), g)
    return every


def _clenshaw_curtis(i):
    """Nodes and weights (of the uniform probability on [-1, 1]) of level i."""
    m = 1 if i == 1 else 2 ** (i - 1) + 1
    if m == 1:
        return np.zeros(1), np.ones(1)
    x = -np.cos(np.pi * np.arange(m) / (m - 1))
    V = np.polynomial.legendre.legvander(x, m - 1).T
    return x, np.linalg.solve(V, np.eye(m)[0])


def _smolyak(d, level):
    from itertools import product

    fine = 2 ** level + 1 if level else 1
    acc = {}
    for lev in product(range(1, level + 2), repeat=d):
        e = level + d - sum(lev)
        if not 0 <= e <= d - 1:
            continue
        rules = [_clenshaw_curtis(i)[1] for i in lev]
        for j in product(*[range(len(w)) for w in rules]):
            key = tuple((fine - 1) // 2 if len(w) == 1 else k * ((fine - 1) // (len(w) - 1)) for k, w in zip(j, rules))
            acc[key] = acc.get(key, 0.0) + (-1) ** e * math.comb(d - 1, e) * math.prod(w[k] for k, w in zip(j, rules))
    keys = sorted(acc)
    grid = -np.cos(np.pi * np.arange(fine) / max(1, fine - 1)) if fine > 1 else np.zeros(1)
    return grid[np.array(keys)], np.array([acc[k] for k in keys])


def _splitmix(seed, c):
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + c.astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _unit(bits):
    return (bits >> np.uint64(11)).astype(np.float64) * 2.0 ** -53


def _rule(spec):
    """Points in [-1, 1], weights, multi-indices and basis of a problem."""
    r, d = spec["rule"], len(spec["dists"])
    if r["kind"] == "gl":
        x, w = np.polynomial.legendre.leggauss(r["n"])
        grids = np.meshgrid(*([x] * d), indexing="ij")
        xi = np.stack([g.reshape(-1) for g in grids], axis=1)
        a = np.ones(1)
        for _ in range(d):
            a = np.multiply.outer(a, w / 2).reshape(-1)
    elif r["kind"] == "smolyak":
        xi, a = _smolyak(d, r["level"])
    else:
        N = r["N"]
        a = np.full(N, 1.0 / N)
        if r["kind"] == "mc":
            xi = 2 * _unit(_splitmix(r["seed"], np.arange(1, N * d + 1))).reshape(N, d) - 1
        elif r["kind"] == "halton":
            xi = np.zeros((N, d))
            for k, p in enumerate((2, 3, 5, 7, 11, 13, 17, 19)[:d]):
                i, f = np.arange(1, N + 1), 1.0 / p
                while i.any():
                    xi[:, k] += f * (i % p)
                    i, f = i // p, f / p
            xi = 2 * xi - 1
        else:
            xi = np.zeros((N, d))
            for k in range(d):
                perm, base = list(range(N)), 2 * N * k
                draws = _splitmix(r["seed"], np.arange(base, base + 2 * N + 1))
                for i in range(N - 1, 0, -1):
                    t = int(draws[i + 1]) * (i + 1) >> 64
                    perm[i], perm[t] = perm[t], perm[i]
                xi[:, k] = 2 * (np.array(perm) + _unit(draws[N + 1:2 * N + 1])) / N - 1
    if r["kind"] not in ("gl", "smolyak"):
        return xi, a, None, None
    alpha = np.array(_multi_indices(d, r["order"]), np.int32)
    one = np.polynomial.legendre.legvander(xi, r["order"]) * np.sqrt(2 * np.arange(r["order"] + 1) + 1)
    phi = np.ones((len(a), len(alpha)))
    for k in range(d):
        phi = phi * one[:, k, alpha[:, k]]
    return xi, a, alpha, phi


def _collide(f, omega):
    """Second-order BGK relaxation of populations less their weights."""
    drho = f.sum(0)
    jx = f[1] - f[3] + f[5] - f[6] - f[7] + f[8]
    jy = f[2] - f[4] + f[5] + f[6] - f[7] - f[8]
    ux, uy = jx / (1 + drho), jy / (1 + drho)
    base = drho - 1.5 * (jx * ux + jy * uy)
    out = torch.empty_like(f)
    for i in range(9):
        eq = base
        if i:
            cj, cu = CX[i] * jx + CY[i] * jy, CX[i] * ux + CY[i] * uy
            eq = base + 3 * cj + 4.5 * cj * cu
        torch.lerp(f[i], WT[i] * eq, omega, out=out[i])
    return out


def _velocity(f):
    rho = 1 + f.sum(0)
    return rho, (f[1] - f[3] + f[5] - f[6] - f[7] + f[8]) / rho, (f[2] - f[4] + f[5] + f[6] - f[7] - f[8]) / rho


def _solve(spec, steps, inputs, dev):
    """Populations (less their weights) after `steps` steps, per sample."""
    nx, ny = spec["nx"], spec["ny"]
    T = lambda v: torch.tensor(v, dtype=torch.float64, device=dev)[:, None, None]  # noqa: E731
    x = torch.arange(nx, dtype=torch.float64, device=dev)[None, None, :]
    y = torch.arange(ny, dtype=torch.float64, device=dev)[None, :, None]
    S = len(inputs["nu"])
    omega = T(1.0 / (3 * inputs["nu"] + 0.5))
    if spec["geometry"] == "tgv":
        if spec.get("init") == "harmonic":
            ax, ay = 4 * math.pi / nx * x, 4 * math.pi / ny * y
            eps = 0.25 * (T(inputs["zeta00"]) * torch.sin(2 * ax) * torch.sin(2 * ay)
                          + T(inputs["zeta01"]) * torch.sin(2 * ax) * torch.cos(2 * ay)
                          + T(inputs["zeta10"]) * torch.cos(2 * ax) * torch.sin(2 * ay)
                          + T(inputs["zeta11"]) * torch.cos(2 * ax) * torch.cos(2 * ay))
            u0, aspect = T(inputs["u0"]) * (1 + eps), 1.0
        else:
            ax, ay = 2 * math.pi / nx * x + T(inputs["phase_x"]), 2 * math.pi / ny * y + T(inputs["phase_y"])
            u0, aspect = T(inputs["u0"]), (ny / nx) ** 2
        ux, uy = -u0 * torch.cos(ax) * torch.sin(ay), u0 * torch.sin(ax) * torch.cos(ay)
        drho = -0.75 * u0 * u0 * (torch.cos(2 * ax) + aspect * torch.cos(2 * ay))
        f = torch.empty((9, S, ny, nx), dtype=torch.float64, device=dev)
        for i in range(9):
            cu = CX[i] * ux + CY[i] * uy
            f[i] = WT[i] * (drho + (1 + drho) * (3 * cu + 4.5 * cu * cu - 1.5 * (ux * ux + uy * uy)))
        for _ in range(steps):
            g = _collide(f, omega)
            for i in range(9):
                f[i] = torch.roll(g[i], (CY[i], CX[i]), (1, 2))
        return f, omega, None
    # channel: walls outside the first and last row, a cylinder, open ends
    ch = _channel(spec, dev)
    up, H, ramp = T(inputs["u_peak"])[:, :, 0], float(ny), spec["ramp"]
    profile = (4 * (y[0, :, 0] + 0.5) * (H - y[0, :, 0] - 0.5) / (H * H))[None, :] * up
    f = torch.zeros((9, S, ny, nx), dtype=torch.float64, device=dev)
    for t in range(1, steps + 1):
        g = _collide(f, omega)
        g[:, :, ch["solid"]] = 0.0
        for i in range(9):
            f[i] = torch.roll(g[i], (CY[i], CX[i]), (1, 2))
            if i:
                f[i] = torch.where(ch["back"][i], g[OPP[i]], f[i])
        for i, (ys, xs, q, yb, xb) in ch["cut"].items():
            k, near = OPP[i], q < 0.5
            f[i][:, ys, xs] = torch.where(near, 2 * q * g[k][:, ys, xs] + (1 - 2 * q) * g[k][:, yb, xb],
                                          g[k][:, ys, xs] / (2 * q) + (1 - 1 / (2 * q)) * g[i][:, ys, xs])
        s = math.sin(math.pi * t / (2 * ramp)) ** 2 if 0 < t < ramp else 1.0
        (_ends_zou_he if spec["xbc"] == "zouhe" else _ends_interpolated)(f, s * profile, omega)
        f[:, :, ch["solid"]] = 0.0
    return f, omega, ch


def _channel(spec, dev):
    """Solid nodes, links that bounce back, and links cut by the circle."""
    nx, ny = spec["nx"], spec["ny"]
    curved = spec.get("cyl_bc") == "bouzidi"
    cx, cy, r = (spec["cyl_x"], spec["cyl_y"], 0.5 * spec["cyl_d"]) if curved else (spec["cx"], spec["cy"],
                                                                                   0.5 * spec["D"])
    Y, X = np.mgrid[0:ny, 0:nx]
    solid = (X - cx) ** 2 + (Y - cy) ** 2 <= r * r
    back, into, cut = {}, {}, {}
    for i in range(1, 9):
        sy, sx = Y - CY[i], X - CX[i]
        wall = (sy < 0) | (sy >= ny)
        inside = ~wall & (sx >= 0) & (sx < nx)
        hit = inside & solid[np.clip(sy, 0, ny - 1), np.clip(sx, 0, nx - 1)] & ~solid
        back[i] = torch.from_numpy((wall | (hit & (not curved)))[None]).to(dev)
        into[OPP[i]] = torch.from_numpy(np.stack(np.nonzero(hit))).to(dev)
        if curved:
            ys, xs = np.nonzero(hit)
            dx, dy, a = xs - cx, ys - cy, CX[i] ** 2 + CY[i] ** 2
            h = (CX[i] * dx + CY[i] * dy) / a
            q = h - np.sqrt(h * h - (dx * dx + dy * dy - r * r) / a)
            cut[i] = [torch.from_numpy(np.asarray(v)).to(dev) for v in (ys, xs, q, ys + CY[i], xs + CX[i])]
    return dict(solid=torch.from_numpy(solid).to(dev), back=back, into=into, cut=cut)


def _ends_zou_he(f, u, omega):
    c = [f[i][:, :, 0] for i in range(9)]
    drho = (c[0] + c[2] + c[4] + 2 * (c[3] + c[6] + c[7]) + u) / (1 - u)
    h, ru = 0.5 * (c[2] - c[4]), (1 + drho) * u
    f[1][:, :, 0], f[5][:, :, 0], f[8][:, :, 0] = c[3] + 2 / 3 * ru, c[7] - h + ru / 6, c[6] + h + ru / 6
    c = [f[i][:, :, -1] for i in range(9)]
    v = c[0] + c[2] + c[4] + 2 * (c[1] + c[5] + c[8])
    h = 0.5 * (c[2] - c[4])
    f[3][:, :, -1], f[7][:, :, -1], f[6][:, :, -1] = c[1] - 2 / 3 * v, c[5] + h - v / 6, c[8] - h - v / 6


def _ends_interpolated(f, u_in, omega):
    inner = {k: _velocity(f[:, :, :, k]) for k in (1, 2, -2, -3)}
    for col, sd in ((0, 1), (-1, -1)):
        c = [f[i][:, :, col] for i in range(9)]
        mid = c[0] + c[2] + c[4]
        if col == 0:
            ux = u_in
            rho = 1 + (mid + 2 * (c[3] + c[6] + c[7]) + ux) / (1 - ux)
        else:
            ux, rho = mid + 2 * (c[1] + c[5] + c[8]), torch.ones_like(mid)
        one, two = (inner[1], inner[2]) if col == 0 else (inner[-2], inner[-3])
        dxux, dxuy = sd * (-3 * ux + 4 * one[1] - two[1]) / 2, sd * (4 * one[2] - two[2]) / 2
        dyux = torch.empty_like(ux)
        dyux[:, 1:-1] = (ux[:, 2:] - ux[:, :-2]) / 2
        dyux[:, 0] = (-3 * ux[:, 0] + 4 * ux[:, 1] - ux[:, 2]) / 2
        dyux[:, -1] = (3 * ux[:, -1] - 4 * ux[:, -2] + ux[:, -3]) / 2
        tau = 1.0 / omega[:, :, 0]
        for i in range(9):
            cu = CX[i] * ux
            eq = rho - 1 + rho * (3 * cu + 4.5 * cu * cu - 1.5 * ux * ux)
            f[i][:, :, col] = WT[i] * (eq - 3 * rho * tau * ((CX[i] ** 2 - 1 / 3) * dxux + CX[i] * CY[i] * (dxuy + dyux)))


def _drag(spec, f, omega, ch, u_peak):
    g = _collide(f, omega)
    F = [0.0, 0.0]
    for k in range(1, 9):
        ys, xs = ch["into"][k]
        out = g[k][:, ys, xs] + WT[k]
        back = out
        if ch["cut"]:
            i = OPP[k]
            _, _, q, yb, xb = ch["cut"][i]
            behind, own = g[k][:, yb, xb] + WT[k], g[i][:, ys, xs] + WT[i]
            back = torch.where(q < 0.5, 2 * q * out + (1 - 2 * q) * behind, out / (2 * q) + (1 - 1 / (2 * q)) * own)
        s = (out + back).sum(1).cpu().numpy()
        F[0], F[1] = F[0] + CX[k] * s, F[1] + CY[k] * s
    U_ref = u_peak * (2 / 3 if spec.get("force_ref") == "mean" else 1.0)
    dia = spec["cyl_d"] if ch["cut"] else spec["D"]
    return {"cd": 2 * F[0] / (U_ref ** 2 * dia), "cl": 2 * F[1] / (U_ref ** 2 * dia)}


def _inputs(spec, xi):
    S = len(xi)
    v = {k: np.full(S, float(spec.get(k, 0.0))) for k in ("nu", "u0", "phase_x", "phase_y", "u_peak", "zeta00",
                                                          "zeta01", "zeta10", "zeta11")}
    for k, (t, lo, hi) in enumerate(spec["dists"]):
        val = lo + (hi - lo) * 0.5 * (xi[:, k] + 1)
        if t == "re":
            v["nu"] = spec["u_peak"] * (2 / 3 if spec.get("force_ref") == "mean" else 1.0) * spec["D"] / val
        else:
            v[t] = val
    return v


def _values(spec, steps, qois):
    """Every sample's value of each quantity of interest: [S, n_out]."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    xi, a, alpha, phi = _rule(spec)
    every = _inputs(spec, xi)
    per = max(1, int(6.0e6 / (spec["nx"] * spec["ny"])))
    got = {q: [] for q in qois}
    for s in range(0, len(xi), per):
        part = {k: v[s:s + per] for k, v in every.items()}
        f, omega, ch = _solve(spec, steps, part, dev)
        rho, ux, uy = _velocity(f)
        if ch is not None:
            for v in (rho, ux, uy):
                v[:, ch["solid"]] = 0.0
        if "cd" in qois or "cl" in qois:
            force = _drag(spec, f, omega, ch, part["u_peak"])
        for q in qois:
            if q == "ke":
                u_ref = spec["u0"] if spec["geometry"] == "tgv" else spec["u_peak"]
                v = 2 / (spec["nx"] * spec["ny"] * u_ref ** 2) * (ux * ux + uy * uy).sum((1, 2))[:, None]
            elif q in ("cd", "cl"):
                v = torch.from_numpy(force[q])[:, None]
            else:
                v = {"vel": lambda: torch.stack((ux, uy), 1), "rho": lambda: rho,
                     "speed": lambda: torch.sqrt(ux * ux + uy * uy)}[q]().reshape(len(rho), -1)
            got[q].append(v)
    return {q: torch.cat(v) for q, v in got.items()}, a, alpha, phi


def _statistics(v, a, alpha, phi):
    dev, S = v.device, len(v)
    if phi is None:
        mean = v.mean(0)
        q = ((v - mean) ** 2).sum(0)
        out = {"mean": mean, "var": q / max(1, S - 1), "var_alt": q / S}
    else:
        w = torch.from_numpy(a).to(dev)
        coeffs = (torch.from_numpy(phi).to(dev) * w[:, None]).T @ v
        out = {"mean": coeffs[0], "var": (coeffs[1:] ** 2).sum(0), "var_alt": (w[:, None] * (v - coeffs[0]) ** 2).sum(0),
               "coeffs": coeffs, "alpha": alpha}
    return {k: x.cpu().numpy() if isinstance(x, torch.Tensor) else x for k, x in out.items()}


def exact(case, seed):
    if case["kind"] == "serve":
        out = []
        for spec in _mix(case, seed):
            q = "ke" if spec["geometry"] == "tgv" else "cd"
            v, a, alpha, phi = _values(spec, spec["steps"], [q])
            st = _statistics(v[q], a, alpha, phi)
            K = 0 if alpha is None else len(alpha)
            out.append(dict(S=len(a), K=K, mean=float(st["mean"][0]), var=float(st["var"][0]),
                            var_alt=float(st["var_alt"][0]), coeffs=st["coeffs"][:, 0] if K else np.zeros(0)))
        return _table(out)
    if case["kind"] == "law":
        law = []
        for k, n in enumerate(("n", "n2")):
            spec, u = _law(case, seed + k, case[n])
            v, _, _, _ = _values(spec, case["steps"], ["speed"])
            law.append(torch.sort((v["speed"] / u).reshape(-1))[0])
        at = torch.sort(torch.cat(law))[0]
        F = [torch.searchsorted(x, at[:-1], right=True).double() / len(x) for x in law]
        return {"w1": float(((F[0] - F[1]).abs() * at.diff()).sum())}
    v, a, alpha, phi = _values(_problem(case, seed), case["steps"], case["qois"].split(","))
    return {q: _statistics(x, a, alpha, phi) for q, x in v.items()}
