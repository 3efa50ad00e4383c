"""Benchmark of the batched LBM-UQ hot path on one MI355X.

One benchmark step is one whole UQ job of the batched-collocation workload
(Taylor-Green vortex 256^2, 4-D uniform inputs, 4^4 = 256 Gauss-Legendre
samples, 5000 LBM steps in FP32 shifted populations, gPC order 3): create
(sampling + equilibrium initialisation on the device), run all samples
together, then the per-sample QoI reduction and the FP64 moments / gPC
projection of the kinetic energy and of the velocity field.

Prints one JSON line: aggregate MLUPS (value), the roofline of the dominant
kernel (the stream-collide step, timed with HIP events on its own stream),
and the FP64 oracle timed on host cores on a bounded sample.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, 8 TB/s
BYTES_PER_POP = {"fp64": 8, "fp32": 4, "fp16s": 2, "bf16s": 2}
KERNEL_SRC = [os.path.join(ROOT, "paper_2508_13867_amd", "csrc", f)
              for f in ("lbm_device.h", "fused_shapes.h", "fused_kernels.hip")]
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic_stream_collide_tgv256_fp32.json")
VALU_FILE = os.path.join(ROOT, "profiles", "valu_k_stepR_tgv256_fp32.json")
VALU_ISSUE_PER_S = 256 * 2.4e9  # one wave64 VALU instruction per CU and cycle


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def kernel_hash():
    h = hashlib.sha256()
    for path in KERNEL_SRC:
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def measured_traffic(kernel_prefix):
    """HBM bytes per step launch from the committed rocprofv3 counter runs,
    if they were taken on the current kernel source and on the kernel
    instance this run launches (its name starts with `kernel_prefix`);
    else None."""
    if not os.path.exists(TRAFFIC_FILE):
        return None
    with open(TRAFFIC_FILE) as f:
        t = json.load(f)
    if t.get("kernel_sha") != kernel_hash():
        return None
    if not any(k.replace("void ", "").startswith(kernel_prefix) for k in t.get("kernel", [])):
        return None
    return t.get("bytes_per_launch")


def measured_valu(kernel_prefix):
    """VALU instructions per step launch from the committed rocprofv3 counter
    run, if taken on the current kernel source and kernel instance; else
    None."""
    if not os.path.exists(VALU_FILE):
        return None
    with open(VALU_FILE) as f:
        t = json.load(f)
    if t.get("kernel_sha") != kernel_hash():
        return None
    if not any(k.replace("void ", "").startswith(kernel_prefix) for k in t.get("kernel", [])):
        return None
    return t


def copy_probe(torch, nbytes=1207959552, reps=10):
    """Device-to-device copy of a buffer the size of one step's slab with
    torch's plain copy kernel: the achievable read+write bandwidth (and the
    counter calibration run for the traffic measurement)."""
    a = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    a.fill_(1.0)
    b.copy_(a)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        b.copy_(a)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / reps
    del a, b
    return 2.0 * nbytes / (ms * 1e-3) / 1e9


def serving(U, W, n_jobs, load, log):
    """The light serving trace (W.serving_trace: vortices 64^2..256^2 and
    channels D 10..20): first the batched server's capacity with every job
    submitted at once, then one seeded Poisson arrival schedule at `load`
    times that capacity replayed through the batched server and through the
    plain one (one job at a time, one sample per launch, no graph; the same
    arithmetic): solves/hour, job latency percentiles (completion -
    arrival), aggregate MLUPS, and the largest relative difference between
    the two modes' moments."""
    trace = W.serving_trace(n_jobs=n_jobs)
    jobs = [spec for _, spec in trace]
    work = sum(s["work"] for s in jobs)
    out = {"jobs": n_jobs, "load": load, "trace_seed": W.SEED, "trace_work_node_updates": work}
    log("bench: serving trace, batched capacity (all jobs at once)")
    res, st = _replay(U, jobs, [0.0] * n_jobs, "batched", 32, log, max_jobs=64)
    cap = work / st["elapsed_s"]
    out["batched_capacity"] = dict(_serving_summary(res, st, [0.0]), node_updates_per_s=round(cap, 1))
    arrivals = W.poisson_arrivals(jobs, cap, load)
    means = {}
    for mode in ("batched", "plain"):
        log(f"bench: serving trace at {load}x the batched capacity, {mode} mode")
        res, st = _replay(U, jobs, arrivals, mode, 32, log, max_jobs=64)
        means[mode] = [(r["mean"], r["var"]) for r in res]
        out[mode] = _serving_summary(res, st, arrivals)
        log(f"bench: {mode}: {out[mode]}")
    diff = 0.0
    for (mb, vb), (mp, vp) in zip(means["batched"], means["plain"]):
        diff = max(diff, abs(mb - mp) / max(abs(mp), 1e-300), abs(vb - vp) / max(abs(vp), 1e-300))
    out["max_rel_diff_batched_vs_plain"] = diff
    out["speedup_solves_per_hour"] = round(out["batched"]["solves_per_hour"] / out["plain"]["solves_per_hour"], 2)
    return out


def _replay(U, jobs, arrivals, mode, budget_gb, log, max_jobs=256):
    """Submit `jobs` at the given arrival times (seconds from the start) to a
    fresh server and wait for all of them: results and server statistics."""
    with U.Server(memory_budget_gb=budget_gb, max_jobs=max_jobs, steps_per_tick=96, mode=mode) as srv:
        t0 = time.perf_counter()
        tickets = []
        for arrival, spec in zip(arrivals, jobs):
            dt = arrival - (time.perf_counter() - t0)
            if dt > 0:
                time.sleep(dt)
            tickets.append(srv.submit(spec))
        results = []
        for k, t in enumerate(tickets):
            results.append(srv.wait(t, 1800))
            if (k + 1) % 50 == 0:
                log(f"bench: serving {mode}: {k + 1} of {len(tickets)} jobs done")
        st = srv.stats()
    return results, st


def _serving_summary(results, st, arrivals):
    lat = sorted(r["latency_s"] for r in results)
    return {"jobs": len(results), "failed": sum(r["status"] != 0 for r in results),
            "solves_per_hour": round(st["solves_per_hour"], 1), "mlups": round(st["mlups"], 1),
            "p50_s": round(st["latency_p50_s"], 4), "p99_s": round(st["latency_p99_s"], 4),
            "mean_latency_s": round(st["latency_mean_s"], 4), "max_latency_s": round(lat[-1], 4),
            "makespan_s": round(st["elapsed_s"], 3), "last_arrival_s": round(max(arrivals), 3),
            "arena_peak_gb": round(st["arena_peak_bytes"] / 2 ** 30, 2)}


def study_serving(U, W, log, n_jobs=200, max_work=5.0e10, loads=(0.8, 1.5), n_plain=12, budget_gb=200):
    """The serving mix at full scale (W.serving_mix: 200 seeded jobs, vortex
    64^2..1024^2, cylinder D 10..40, 1..4 inputs, 5..256 collocation nodes
    or 256..4096 Monte Carlo samples, FP32, at most max_work node updates per
    job). (1) Batched capacity: every job submitted at once. (2) Poisson
    arrivals at 0.8x and 1.5x that capacity: latency percentiles, solves per
    hour, aggregate MLUPS. (3) Plain mode (one job at a time, one sample per
    launch, no graph) against batched on the same subset of jobs submitted at
    once, with their results compared bit for bit."""
    jobs = W.serving_mix(n_jobs, max_work=max_work)
    work = sum(j["work"] for j in jobs)
    out = {"jobs": n_jobs, "max_work_per_job": max_work, "trace_seed": W.SEED, "work_node_updates": work,
           "budget_gb": budget_gb}
    log(f"bench: serving mix of {n_jobs} jobs, {work:.3g} node updates: capacity run")
    res, st = _replay(U, jobs, [0.0] * n_jobs, "batched", budget_gb, log)
    cap = work / st["elapsed_s"]
    out["capacity"] = dict(_serving_summary(res, st, [0.0]), node_updates_per_s=cap)
    log(f"bench: capacity {out['capacity']}")
    ref = {j["name"]: (r["mean"], r["var"]) for j, r in zip(jobs, res)}
    for load in loads:
        arr = W.poisson_arrivals(jobs, cap, load)
        res, st = _replay(U, jobs, arr, "batched", budget_gb, log)
        out[f"load_{load}"] = _serving_summary(res, st, arr)
        # a job's result does not depend on what ran beside it
        out[f"load_{load}"]["bitwise_same_as_capacity_run"] = all(
            (r["mean"], r["var"]) == ref[j["name"]] for j, r in zip(jobs, res))
        log(f"bench: load {load}: {out[f'load_{load}']}")
    # plain vs batched on the first jobs whose one-sample-per-launch run is
    # short (launch-bound: about 5 us per launch, or the lattice's bytes at
    # 5 TB/s)
    est = [j["work"] / (j["nx"] * j["ny"]) * max(5e-6, j["nx"] * j["ny"] * 36 / 5e12) for j in jobs]
    sub = [j for j, e in zip(jobs, est) if e < 6.0][:n_plain]
    sw = sum(j["work"] for j in sub)
    out["plain_subset"] = {"jobs": [j["name"] for j in sub], "work_node_updates": sw}
    pres = {}
    for mode in ("plain", "batched"):
        log(f"bench: subset of {len(sub)} jobs, {mode}")
        res, st = _replay(U, sub, [0.0] * len(sub), mode, budget_gb, log)
        out["plain_subset"][mode] = _serving_summary(res, st, [0.0])
        pres[mode] = [(r["mean"], r["var"]) for r in res]
    out["plain_subset"]["bitwise_batched_equals_plain"] = pres["plain"] == pres["batched"]
    out["plain_subset"]["speedup_solves_per_hour"] = round(
        out["plain_subset"]["batched"]["solves_per_hour"] / out["plain_subset"]["plain"]["solves_per_hour"], 2)
    return out


def study_precision(U, W, log, oracle_samples=8):
    """Monte Carlo workload (128^2 vortex, 4-D inputs, 4096 samples, 2000
    steps) in FP64, FP32, FP16- and BF16-storage: throughput and roofline per
    precision, the error of E[K] and Var[K] against the FP64 run (itself
    re-checked sample by sample against the FP64 oracle), and the Monte Carlo
    rate: RMS error of the mean over disjoint groups of N samples against a
    6^4-node Gauss-Legendre collocation reference."""
    import numpy as np

    import oracle as O

    base = dict(W.TGV_MC)
    out = {"workload": base["name"], "runs": {}}
    ke = {}
    for prec in ("fp64", "fp32", "fp16s", "bf16s"):
        spec = dict(base, precision=prec)
        tune = U.autotune(spec, steps=20)
        with U.Job(spec) as job:
            inf = job.info()
            ms = job.run_timed(spec["steps"])
            launches = job.info().step_launches
            st = job.moments("ke")
            ke[prec] = job.qoi_samples("ke")[:, 0]
        nodes = job.S * spec["nx"] * spec["ny"]
        bpn = 18 * BYTES_PER_POP[prec]  # per node per launch (read + write once)
        launch_ms = ms / launches
        out["runs"][prec] = {"mean": st["mean"][0], "var": st["var"][0],
                             "mlups": round(nodes * spec["steps"] / (ms * 1e-3) / 1e6, 1),
                             "gbs": round(nodes * bpn / (launch_ms * 1e-3) / 1e9, 1),
                             "frac_hbm": round(nodes * bpn / (launch_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
                             "bytes_per_node_update": round(bpn * launches / spec["steps"], 3),
                             "steps_per_launch": inf.fused or 1, "layout": {1: "aa", 2: "ab"}[inf.layout],
                             "scale_exp": inf.scale_exp, "tuned_gbs": round(tune["gbs"], 1)}
        log(f"bench: precision {prec}: {out['runs'][prec]}")
    r64 = out["runs"]["fp64"]
    for prec, r in out["runs"].items():
        r["err_mean_vs_fp64"] = abs(r["mean"] - r64["mean"]) / abs(r64["mean"])
        r["err_var_vs_fp64"] = abs(r["var"] - r64["var"]) / abs(r64["var"])
        r["err_samples_rel_l2_vs_fp64"] = float(np.linalg.norm(ke[prec] - ke["fp64"]) / np.linalg.norm(ke["fp64"]))
    # the FP64 run against the oracle, sample by sample
    pick = list(range(0, 4096, 4096 // oracle_samples))[:oracle_samples]
    log(f"bench: oracle re-solves samples {pick}")
    ref = O.run_problem(base, samples=pick, qois=["ke"])
    err = float(np.linalg.norm(ke["fp64"][pick] - ref["samples"]["ke"]) / np.linalg.norm(ref["samples"]["ke"]))
    out["fp64_vs_oracle_rel_l2_sampled"] = err
    out["oracle_samples"] = pick
    # Monte Carlo rate against a collocation reference
    gl = dict(base, precision="fp64", rule=dict(kind="gl", n=6, order=5), name="tgv128_gl6x4")
    with U.Job(gl) as job:
        job.run(gl["steps"])
        ref_mean = job.moments("ke")["mean"][0]
    rates = []
    for N in (16, 32, 64, 128, 256):  # at least 16 disjoint groups each
        groups = ke["fp64"][: 4096 // N * N].reshape(-1, N).mean(axis=1)
        rates.append((N, float(np.sqrt(np.mean((groups - ref_mean) ** 2)))))
    slope = float(np.polyfit(np.log([n for n, _ in rates]), np.log([e for _, e in rates]), 1)[0])
    out["mc_reference_gl6x4_mean"] = ref_mean
    out["mc_rms_error_by_N"] = rates
    out["mc_rate_slope"] = slope
    return out


def study_samplers(U, W, log):
    """Convergence of E[K] and Var[K] (128^2 vortex, 4-D inputs, 2000 steps,
    FP32) for Monte Carlo, Halton quasi Monte Carlo, Latin hypercube, Smolyak
    sparse grids and tensor Gauss-Legendre collocation, against a 6^4-node
    tensor Gauss-Legendre reference (the analogue of the paper's MC / QMC /
    SC-gPC comparisons)."""
    base = dict(W.TGV_MC)
    runs = []

    def run(rule, label):
        spec = dict(base, rule=rule, name=label)
        with U.Job(spec) as job:
            ms = job.run_timed(spec["steps"])
            st = job.moments("ke")
            S = job.S
        r = {"label": label, "rule": rule, "samples": S, "mean": st["mean"][0], "var": st["var"][0],
             "ms": round(ms, 2)}
        log(f"bench: samplers {r}")
        return r

    ref = run(dict(kind="gl", n=6, order=5), "gl6")
    for N in (64, 256, 1024, 4096):
        runs.append(run(dict(kind="mc", N=N, seed=W.SEED), f"mc{N}"))
        runs.append(run(dict(kind="halton", N=N), f"halton{N}"))
        runs.append(run(dict(kind="lhs", N=N, seed=W.SEED), f"lhs{N}"))
    for lvl in (1, 2, 3, 4):
        runs.append(run(dict(kind="smolyak", level=lvl, order=min(lvl, 3)), f"smolyak{lvl}"))
    for n in (2, 3, 4, 5):
        runs.append(run(dict(kind="gl", n=n, order=n - 1), f"gl{n}"))
    for r in runs:
        r["err_mean"] = abs(r["mean"] - ref["mean"]) / abs(ref["mean"])
        r["err_var"] = abs(r["var"] - ref["var"]) / abs(ref["var"])
    return {"workload": "tgv128 4-D inputs, 2000 steps, FP32", "reference": ref, "runs": runs}


def study_cylinder(U, W, log, oracle_samples=1):
    """The cylinder workload at full size (440 x 82, 8 x 8 collocation,
    20000 steps, FP32): C_D and C_L statistics and gPC coefficients, with one
    sample re-solved by the FP64 oracle over the full 20000 steps."""
    import numpy as np

    import oracle as O

    spec = dict(W.CYLINDER_FP32)
    tune = U.autotune(spec, steps=40)
    with U.Job(spec) as job:
        ms = job.run_timed(spec["steps"])
        cd, cl = job.moments("cd"), job.moments("cl")
        cd_s = job.qoi_samples("cd")[:, 0]
        cl_s = job.qoi_samples("cl")[:, 0]
        nodes = job.S * spec["nx"] * spec["ny"]
    out = {"workload": spec["name"], "tuned": tune, "ms": ms,
           "mlups": round(nodes * spec["steps"] / (ms * 1e-3) / 1e6, 1),
           "cd": {"mean": cd["mean"][0], "std": float(np.sqrt(cd["var"][0])), "var_quad": cd["var_alt"][0],
                  "coeffs_first6": cd["coeffs"][:6, 0].tolist()},
           "cl": {"mean": cl["mean"][0], "std": float(np.sqrt(cl["var"][0]))}}
    pick = [27][:oracle_samples]
    log(f"bench: oracle re-solves cylinder sample {pick} over {spec['steps']} steps")
    ref = O.run_problem(spec, samples=pick, qois=["cd", "cl"])
    out["oracle_samples"] = pick
    out["cd_sample_rel_err_vs_oracle"] = float(abs(cd_s[pick] - ref["samples"]["cd"]).max() /
                                               abs(ref["samples"]["cd"]).max())
    out["cl_sample_abs_err_vs_oracle"] = float(abs(cl_s[pick] - ref["samples"]["cl"]).max())
    out["cd_sample_oracle"] = ref["samples"]["cd"].tolist()
    return out


def study_wasserstein(U, W, log, prec="fp32", ns=(8, 16, 32, 64, 128), n_ref=256, fracs=(0.2, 0.4, 0.6, 0.8, 1.0),
                      chunk=40000):
    """Wasserstein convergence of the numerical statistical solutions of the
    four-dimensional perturbed vortex: for each resolution n (N = n samples,
    Table tab:simulation_parameters units, FP32) and each checkpoint t =
    frac T_max, W_1 between the law of |u| (all nodes of all samples, in
    physical units |u| / u_lat) at n and at the reference resolution, with
    the observed rate of decay in n. A re-run of n = 128 in the other
    precision measures what the storage precision alone moves the statistic
    by. The initial field is invariant under a shift by half the period in
    x; `asym` is the largest departure from that symmetry, max |u(x + n/2, y)
    - u(x, y)| / u_lat over all samples: exact arithmetic keeps it at zero,
    so its growth is symmetry breaking seeded by rounding."""
    import numpy as np

    def asym(job, n, u_lat):
        v = job.qoi_samples("vel").reshape(job.S, 2, n, n)
        return float(np.abs(np.roll(v, -(n // 2), axis=3) - v).max() / u_lat)

    res = {}
    for n in ns + (n_ref,):
        u = U.tgv_units(n, 1.6 / n, 40.0 * n)
        res[n] = {"units": u, "job": U.Job(W.tgv4d(n, u, precision=prec)), "done": 0, "ms": 0.0}
    out = {"workload": f"tgv4d, n = 8..128 against 256, N = n MC samples, T_max = 100, {prec.upper()}",
           "precision": prec, "units": {n: r["units"] for n, r in res.items()}, "checkpoints": []}
    try:
        for f in fracs:
            t = f * W.TGV4D_T_MAX
            for n, r in res.items():
                target = int(round(t / r["units"]["dt"]))
                while r["done"] < target:
                    k = min(chunk, target - r["done"])
                    r["ms"] += r["job"].run_timed(k)
                    r["done"] += k
                    if n == n_ref:
                        log(f"bench: tgv4d n={n} step {r['done']} of {target} (t = {t:g})")
            ref = res[n_ref]
            cp = {"t": t, "frac": f, "steps": {n: r["done"] for n, r in res.items()}, "w1": {}}
            for n in ns:
                cp["w1"][n] = U.wasserstein1(res[n]["job"], ref["job"], "speed", 1.0 / res[n]["units"]["u_lat"],
                                             1.0 / ref["units"]["u_lat"])
            cp["mean_speed_ref"] = float(np.mean(ref["job"].moments("speed")["mean"]) / ref["units"]["u_lat"])
            cp["asym"] = {n: asym(r["job"], n, r["units"]["u_lat"]) for n, r in res.items()}
            x, y = np.log(np.array(ns, float)), np.log(np.array([cp["w1"][n] for n in ns]))
            cp["rate_all"] = float(-np.polyfit(x, y, 1)[0])
            cp["rate_last3"] = float(-np.polyfit(x[-3:], y[-3:], 1)[0])
            log(f"bench: tgv4d t={t:g} W1 {cp['w1']} rate {cp['rate_all']:.2f} (last three {cp['rate_last3']:.2f})")
            out["checkpoints"].append(cp)
        for n, r in res.items():
            nodes = r["job"].S * n * n
            out.setdefault("mlups", {})[n] = round(nodes * r["done"] / (r["ms"] * 1e-3) / 1e6, 1)
        # what the storage precision alone changes at n = 128, T_max
        n = 128
        r = res[n]
        other = "fp64" if prec != "fp64" else "fp32"
        with U.Job(W.tgv4d(n, r["units"], precision=other)) as jo:
            done = 0
            while done < r["done"]:
                k = min(chunk, r["done"] - done)
                jo.run(k)
                done += k
                log(f"bench: tgv4d n={n} {other} step {done} of {r['done']}")
            out["fp32_vs_fp64_w1_n128"] = U.wasserstein1(r["job"], jo, "speed", 1.0 / r["units"]["u_lat"],
                                                         1.0 / r["units"]["u_lat"])
            out[f"asym_n128_{other}"] = asym(jo, n, r["units"]["u_lat"])
    finally:
        for r in res.values():
            r["job"].close()
        for r in res.values():
            del r["job"]
    return out


def study_cylinder_paper(U, W, log, steps=40000, n_mc=1000):
    """The paper's cylinder set-up (22D x 4D, D = 20, interpolated circle,
    finite-difference inlet/outlet, u_in = u(1 + 0.2 xi), Re = 20 on the mean
    inflow, FP32): mean and standard deviation of C_D by Monte Carlo, Halton
    quasi Monte Carlo and Gauss-Legendre SC-gPC, and the deterministic value,
    next to the paper's Table tab:uq_results; the drag history of the
    deterministic run; a resolution study (D = 10, 20, 40) of the
    deterministic drag for the interpolated and the half-way/Zou-He
    boundaries; and the literal reading (peak velocity in Re and C_D)."""
    import numpy as np

    base = dict(W.CYLINDER_PAPER_FP32, steps=steps)
    paper = {"mc": (5.66731, 0.34896), "qmc": (5.67270, 0.34890), "sc": (5.67261, 0.34888),
             "deterministic": (5.63208, None)}
    out = {"workload": base["name"] + f", {steps} steps", "paper_table": paper, "runs": {}}

    def run(spec, label, checkpoints=()):
        with U.Job(spec) as job:
            hist, done, ms = [], 0, 0.0
            for c in list(checkpoints) + [spec["steps"]]:
                if c > done:
                    ms += job.run_timed(c - done)
                    done = c
                if c in checkpoints:
                    hist.append((c, float(job.qoi_samples("cd")[:, 0].mean())))
            st = job.moments("cd")
            cd = job.qoi_samples("cd")[:, 0]
            cl = job.qoi_samples("cl")[:, 0]
            nodes = job.S * spec["nx"] * spec["ny"]
        r = {"samples": int(cd.size), "mean": float(st["mean"][0]), "std": float(np.sqrt(st["var"][0])),
             "cl_max_abs": float(np.abs(cl).max()), "ms": round(ms, 1),
             "mlups": round(nodes * spec["steps"] / (ms * 1e-3) / 1e6, 1)}
        if hist:
            r["history"] = hist
        log(f"bench: cylinder paper {label} {r}")
        out["runs"][label] = r
        return r

    run(W.scaled(base, rule=dict(kind="gl", n=1, order=0)), "deterministic",
        checkpoints=(5000, 10000, 20000, 30000))
    run(base, "sc")
    run(W.scaled(base, rule=dict(kind="mc", N=n_mc, seed=W.SEED)), "mc")
    run(W.scaled(base, rule=dict(kind="halton", N=n_mc)), "qmc")
    # resolution study of the deterministic drag (lattice velocity fixed, so
    # nu and the step count scale with D)
    for D in (10, 20, 40):
        for scheme in ("interp", "halfway"):
            f = D / 20
            spec = W.scaled(base, name=f"cyl_D{D}_{scheme}", nx=22 * D, ny=4 * D, cyl_x=2.0 * D,
                            cyl_y=(4 * D - 1) / 2, cyl_d=float(D), nu=0.04 * f, steps=int(steps * f),
                            ramp=int(base["ramp"] * f), rule=dict(kind="gl", n=1, order=0))
            if scheme == "halfway":
                spec = W.scaled(spec, cyl_bc="halfway", xbc="zouhe", D=D, cx=2 * D, cy=2 * D)
            run(spec, f"resolution_D{D}_{scheme}")
    # the literal reading: peak inflow in Re and in C_D
    run(W.scaled(base, nu=0.06, force_ref="peak", rule=dict(kind="gl", n=1, order=0)), "literal_peak_reading")
    # sensitivity of the deterministic drag to set-up details the paper
    # leaves open: the channel height (4.1 D instead of 4 D, circle centred)
    # and the lattice Mach number (mean inflow 0.03 instead of 0.04, nu and
    # the step count scaled to keep Re = 20 and the physical time)
    det = dict(rule=dict(kind="gl", n=1, order=0))
    run(W.scaled(base, ny=82, cyl_y=40.5, **det), "height_4.1D")
    run(W.scaled(base, u_peak=0.045, nu=0.03, steps=int(steps * 4 / 3), ramp=int(base["ramp"] * 4 / 3),
                 dists=[("u_peak", 0.036, 0.054)], **det), "mach_0.75x")
    return out


def _oracle_one(args):
    """One oracle sample (a worker of the sample-parallel CPU baseline)."""
    import oracle as O

    spec, xi_row, steps = args
    O.solve_sample(spec, O.sample_params(spec, xi_row), steps=steps)
    return 0


def cpu_baseline(spec, n_samples=4, lbm_steps=300, max_cores=16):
    """The FP64 oracle on the full lattice of the workload for a few samples
    and steps: single-threaded (about 4 s), then the paper's sample-level
    parallelism, one sample per process on every host core available to this
    process (at most max_cores; about 1 s). Runs before the GPU is touched,
    so the worker processes are plain forks of a process without device state."""
    import multiprocessing as mp

    import oracle as O

    O.build()
    xi, a = O.sample_set(spec)
    cells = spec["nx"] * spec["ny"]
    t0 = time.perf_counter()
    for j in range(n_samples):
        O.solve_sample(spec, O.sample_params(spec, xi[j]), steps=lbm_steps)
    dt1 = time.perf_counter() - t0
    single = n_samples * cells * lbm_steps / dt1 / 1e6
    cores = max(1, min(max_cores, len(os.sched_getaffinity(0))))
    work = [(spec, xi[j % len(xi)], lbm_steps) for j in range(cores)]
    with mp.get_context("fork").Pool(cores) as pool:
        pool.map(_oracle_one, [(spec, xi[0], 1)] * cores)  # start the workers first
        t0 = time.perf_counter()
        pool.map(_oracle_one, work, chunksize=1)
        dtp = time.perf_counter() - t0
    par = cores * cells * lbm_steps / dtp / 1e6
    return {"value": round(par, 3), "unit": "MLUPS", "cores": cores, "kind": "oracle",
            "sample": f"{cores} samples x {lbm_steps} steps on the full {spec['nx']}x{spec['ny']} lattice, one "
                      f"FP64 oracle process per core (sample-level parallelism), {dtp:.1f} s",
            "single_core_mlups": round(single, 3),
            "single_core_sample": f"{n_samples} samples x {lbm_steps} steps, one thread, {dt1:.1f} s"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3, help="timed UQ jobs")
    ap.add_argument("--warmup", type=int, default=1, help="untimed UQ jobs")
    ap.add_argument("--workload", default="tgv256_fp32_gl4x4")
    ap.add_argument("--lbm-steps", type=int, default=None, help="override LBM steps per job")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--copy-probe", action="store_true", help="only run the copy-bandwidth probe")
    ap.add_argument("--tune-steps", type=int, default=40, help="steps per candidate of the launch-shape tuner")
    ap.add_argument("--no-serving", action="store_true", help="skip the serving-trace comparison")
    ap.add_argument("--study", choices=["precision", "cylinder", "samplers", "wasserstein", "cylinder_paper", "serving"],
                    default=None,
                    help="run a measurement study instead of the benchmark and print its JSON")
    ap.add_argument("--study-precision", default="fp32", choices=["fp64", "fp32"],
                    help="storage precision of the wasserstein study")
    ap.add_argument("--serving-jobs", type=int, default=24)
    ap.add_argument("--serving-load", type=float, default=1.5, help="offered load of the serving trace, "
                    "as a multiple of the batched capacity measured first")
    ap.add_argument("--no-tune", action="store_true",
                    help="skip tuning (shapes then come from UQ_TUNE_CACHE or the defaults)")
    args = ap.parse_args()

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on one GPU only; the multi-GPU layout (sample sharding with one "
              "all-reduce of the FP64 moment partial sums) is described in the design notes but not run.",
              file=sys.stderr)
        sys.exit(2)

    import torch

    import paper_2508_13867_amd as U
    from paper_2508_13867_amd import workloads as W

    spec = dict(W.WORKLOADS[args.workload])
    if args.lbm_steps:
        spec["steps"] = args.lbm_steps
    prec = spec["precision"]
    cells = spec["nx"] * spec["ny"]
    cpu = None
    if not args.no_cpu_baseline and args.study is None and not args.copy_probe:
        log("bench: CPU oracle baseline (before any device work)")
        cpu = cpu_baseline(spec)
        log(f"bench: CPU oracle {cpu}")
    torch.cuda.init()
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    copy_gbs = copy_probe(torch)
    log(f"bench: device copy {copy_gbs:.0f} GB/s")
    if args.copy_probe:
        print(json.dumps({"copy_gbs": round(copy_gbs, 1)}), flush=True)
        return
    if args.study == "precision":
        print(json.dumps(study_precision(U, W, log)), flush=True)
        return
    if args.study == "cylinder":
        print(json.dumps(study_cylinder(U, W, log)), flush=True)
        return
    if args.study == "samplers":
        print(json.dumps(study_samplers(U, W, log)), flush=True)
        return
    if args.study == "cylinder_paper":
        print(json.dumps(study_cylinder_paper(U, W, log)), flush=True)
        return
    if args.study == "serving":
        print(json.dumps(study_serving(U, W, log)), flush=True)
        return
    if args.study == "wasserstein":
        print(json.dumps(study_wasserstein(U, W, log, prec=args.study_precision)), flush=True)
        return

    tune = None
    if not args.no_tune:
        log("bench: tuning the launch shape")
        tune = U.autotune(spec, steps=args.tune_steps)
        log(f"bench: tuned {tune}")
    launch = {}

    def one_job(timed_kernel):
        job = U.Job(spec, device=0)
        inf = job.info()
        launch.update(layout={1: "aa", 2: "ab"}[inf.layout], cpt=inf.cpt, nt_store=inf.nt_store,
                      plane_pad=inf.plane_pad, bx=inf.bx, fused_steps=inf.fused, fused_rows=inf.fused_rows,
                      fused_window=inf.fused_window, device_bytes=inf.device_bytes)
        ms = job.run_timed(spec["steps"]) if timed_kernel else None
        if not timed_kernel:
            job.run(spec["steps"])
        launches = job.info().step_launches
        job.moments("ke")
        job.moments("vel")
        S = job.S
        job.close()
        return S, ms, launches

    log(f"bench: workload {spec['name']} warmup {args.warmup} jobs")
    for _ in range(args.warmup):
        one_job(False)
    torch.cuda.synchronize()

    log(f"bench: timing {args.steps} jobs")
    kernel_ms = []
    t0 = time.perf_counter()
    S = 0
    n_launch = []
    for k in range(args.steps):
        S, ms, nl = one_job(True)
        kernel_ms.append(ms)
        n_launch.append(nl)
        log(f"bench: job {k} done, {nl} step launches, {ms:.1f} ms")
    torch.cuda.synchronize()
    t1 = time.perf_counter()

    wall = t1 - t0
    updates = args.steps * S * cells * spec["steps"]
    mlups = updates / wall / 1e6
    ms_per_job = wall / args.steps * 1e3

    # dominant kernel: every step launch (single or fused) reads the 9
    # populations of each of the S * cells nodes once and writes them once;
    # a fused launch advances them `fused_steps` steps
    bpn = 18 * BYTES_PER_POP[prec]
    launches = sum(n_launch)
    per_launch_ms = sum(kernel_ms) / launches
    alg_bytes = S * cells * bpn
    achieved = alg_bytes / (per_launch_ms * 1e-3) / 1e9
    nfuse = launch.get("fused_steps", 0) or 1
    pcode = {"fp64": 0, "fp32": 1, "fp16s": 2, "bf16s": 3}[prec]
    if nfuse > 1 and launch.get("fused_window") == 2:
        kprefix = f"uqi::k_stepR<{pcode}, {nfuse}, "
    elif nfuse > 1 and launch.get("fused_window"):
        kprefix = f"uqi::k_stepW<{pcode}, {nfuse}, "
    elif nfuse > 1:
        kprefix = f"uqi::k_stepN<{pcode}, {launch.get('fused_rows')}, {nfuse}>"
    else:
        kprefix = "uqi::k_step<"
    traffic = measured_traffic(kprefix)
    valu = measured_valu(kprefix)
    hbm = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
           "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic, "bytes_per_launch": alg_bytes,
           "bytes_per_node_update": round(bpn / nfuse, 3), "copy_gbs": round(copy_gbs, 1),
           "frac_of_copy": round(achieved / copy_gbs, 4)}
    common = {"kernel": ({0: f"uqi::k_stepN<..., N={nfuse}>", 1: f"uqi::k_stepW<..., N={nfuse}>",
                          2: f"uqi::k_stepR<..., N={nfuse}>"}[launch.get("fused_window") or 0]
                         if nfuse > 1 else "uqi::k_step"),
              "updates_per_node_per_launch": nfuse, "launches": launches, "launch_ms": round(per_launch_ms, 5)}
    roof = dict(hbm, **common)
    if valu is not None:
        # the other bound of the fused kernels: VALU instruction issue. Its
        # peak is 256 CUs x 2.4 GHz x 64 lanes (one wave64 VALU instruction
        # per CU and cycle; packed FP32, which the datasheet's 157.3 TFLOP/s
        # counts, is not used). The line reports the tighter of the two.
        lane_ops = valu["valu_insts_per_launch"] * 64.0
        alu_achieved = lane_ops / (per_launch_ms * 1e-3) / 1e12
        alu_peak = VALU_ISSUE_PER_S * 64.0 / 1e12
        alu = {"bound": "alu", "achieved": round(alu_achieved, 3), "peak": round(alu_peak, 3),
               "unit": "T VALU lane-ops/s", "frac": round(alu_achieved / alu_peak, 4), "traffic": traffic,
               "lane_ops_per_launch": lane_ops, "lane_ops_per_node_update": round(valu["valu_lane_ops_per_update"], 2)}
        if alu["frac"] > hbm["frac"]:
            roof = dict(alu, **common, hbm=hbm)
        else:
            roof = dict(hbm, **common, alu=alu)

    out = {
        "metric": "aggregate MLUPS & % HBM peak; UQ solves/hr + p50/p99 latency vs plain",
        "value": round(mlups, 1),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_job, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {"fp64": "f64", "fp32": "f32", "fp16s": "f16-storage/f32", "bf16s": "bf16-storage/f32"}[prec],
        "data": "synthetic",
        "config": {"workload": spec["name"], "nx": spec["nx"], "ny": spec["ny"], "samples": S,
                   "lbm_steps": spec["steps"], "rule": spec["rule"], "precision": prec,
                   "moments": "FP64 compensated, KE + velocity field", "launch": launch},
        "roofline": roof,
        "uq_solves_per_hour": round(3600.0 / (wall / args.steps), 1),
        "hbm_frac_of_peak": hbm["frac"],
    }
    if not args.no_serving:
        out["serving"] = serving(U, W, args.serving_jobs, args.serving_load, log)
        out["uq_solves_per_hour_serving"] = out["serving"]["batched"]["solves_per_hour"]
        out["p50_s"] = out["serving"]["batched"]["p50_s"]
        out["p99_s"] = out["serving"]["batched"]["p99_s"]
    if cpu is not None:
        out["cpu_baseline"] = cpu
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
