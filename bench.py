#!/usr/bin/env python3
"""Benchmark of the screened-interaction path on one MI355X.

Default workload (`n2000`): W(omega) per second for one molecule of exactly
2000 products (the 40-atom chain truncated to its first 2000 products) on the
1024-point mesh.  One step = the whole path: pair vertex, mesh bins, exact
int64 histogram, FFT chi0 on all 1024 mesh points (gw_build_chi0), then
W(omega) = (1 - v chi0)^{-1} v on all 1024 points (gw_solve_W: 513 factorised,
the rest by the conjugate mirror).  The `_A` forms take the same path with A =
1 - v chi0 formed at the FFT from v a0 (gw_build_A: one real product by v per
spectral bin instead of one complex product per solved frequency), then W
from A (gw_solve_W_A).  Inputs are resident in HBM before the timed region.
The precision forms are timed in turn (FP64; FP32 LU + FP64 residual
refinement; the same with split-BF16 trailing updates; each on either route);
`value` is the fastest form that meets the 1e-6 error target relative to the
FP64 chi0-route result.

Other workloads (one JSON line each, same keys):
  c1    the 40-atom chain with all of its products
  c2    120-atom cluster, v compressed to its top-1500 subspace, 2048 points
  c2pair  the same cluster in the paper's own pair subspace (k = 256)
  n2000_2w  the 2000-product molecule with two spectral windows (256 fine
        points over |omega| < 0.5 Ha, 256 coarse ones over |omega| < 4 Ha)
  n2000_time  the 2000-product molecule, a0 by the paper's time-domain route
  n2000_sigma  the same carried through to the GW self-energy on all points
  c3    64 chain molecules (8..80 atoms, 512 points) as recorded hipGraph
        batches, solved in place (A = 1 - v chi0 formed from v a0 in each
        molecule's buffer, then W over it)
  c4    serving: Poisson arrivals at 20/s for 60 s (overloaded), then a
        labelled below-capacity run

    python bench.py [--steps K] [--warmup W] [--gpus 1] [--workload n2000]
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
N_PROD = 2000
PEAK_FP64 = 78.6e12
PEAK_FP32 = 157.3e12
FORMS = {"fp64": 0, "fp32_ir": 1, "bf16x_ir": 2}  # gw_precision values
# the form the committed profiles were taken on (the default headline form),
# and the step it times
PROFILE_FORM = "fp64_A"
PROFILE_STEP = "FP64 step (A = 1 - v chi0 from v a0 + W solve)"


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def solve_flops(n, n_solved, n_ir=0, mixed=False, form_a=True):
    """Algorithmic flops of the W solve per solved frequency.  FP64: A = 1 -
    v chi0 4N^3, LU 8/3 N^3, forward substitution with N right-hand sides 4N^3,
    back substitution of the lower triangle of the symmetric W 4/3 N^3
    (sum over rows r of (r + 1)(N - 1 - r) complex multiply-adds).  Mixed:
    low-precision LU and full solves (8N^3), and per refinement step an FP64
    residual 8N^3 and a low-precision solve 8N^3.  form_a = False: A is an
    input (formed with chi0 from v a0), no 4N^3 product."""
    n3 = float(n) ** 3
    fa = 4.0 if form_a else 0.0
    if not mixed:
        return {"fp64": n_solved * (fa + 8.0 / 3 + 4 + 4.0 / 3) * n3, "fp32": 0.0}
    return {"fp64": n_solved * (fa + 8 * n_ir) * n3, "fp32": n_solved * (8.0 / 3 + 8 * (1 + n_ir)) * n3}


def solve_roofline(n, n_solved, t_solve, n_ir, mixed, form_a=True):
    fl = solve_flops(n, n_solved, n_ir, mixed, form_a)
    t_roof = fl["fp64"] / PEAK_FP64 + fl["fp32"] / PEAK_FP32
    total = fl["fp64"] + fl["fp32"]
    achieved = total / t_solve / 1e12
    peak = total / t_roof / 1e12
    return achieved, peak


def blas_threads():
    try:
        from threadpoolctl import threadpool_info

        return max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        return os.cpu_count()


def cpu_baseline(mol, grid, budget_s=20.0):
    """Oracle on the host cores over a bounded sample, scaled to whole-job
    delivered W(omega)/s.  The oracle uses the same conjugate mirror as the
    GPU (W(-omega) = W(omega)*, exact for the retarded response on the
    symmetric mesh), so it pays chi0 and a LAPACK solve at the same N/2 + 1
    frequencies: T = T_pairs + T_hist + (N/2 + 1) (T_chi0(w) + T_W(w))."""
    sys.path.insert(0, HERE)
    import oracle as o

    t0 = time.perf_counter()
    P = o.pair_vectors(mol)
    t_pairs = time.perf_counter() - t0
    d = grid.domega
    m, fr = o.pair_bins(mol.eig, mol.n_occ, d)
    nhb = o.hist_bins(mol.eig, grid.n_omega, d)
    s = o.frac_bits(P, mol.n_pairs)
    n = mol.n_prod
    n_upper = n * (n + 1) // 2
    rng = np.random.default_rng(0)
    n_samp = 4000
    idx = np.sort(rng.choice(n_upper, size=n_samp, replace=False))
    iu, ju = np.triu_indices(n)
    t0 = time.perf_counter()
    H, _ = o.histogram_c(P, m, fr, s, nhb, iu[idx], ju[idx])
    t_hist = (time.perf_counter() - t0) * n_upper / n_samp
    # chi0 at one frequency for the sampled entries, scaled to all entries
    t0 = time.perf_counter()
    o.chi0_from_hist(H, s, grid.n_omega, grid.omega_min, grid.omega_max, grid.eps, js=[grid.n_omega // 2 + 40])
    t_chi = (time.perf_counter() - t0) * n_upper / n_samp
    # dense solve at full size, a few frequencies (cost independent of omega)
    rs = np.random.default_rng(1)
    chi = (rs.standard_normal((n, n)) + 1j * rs.standard_normal((n, n))) * 1e-3
    chi = chi + chi.T
    ts = []
    t_start = time.perf_counter()
    while len(ts) < 3 and time.perf_counter() - t_start < budget_s:
        t0 = time.perf_counter()
        o.screened_W(mol.v, chi)
        ts.append(time.perf_counter() - t0)
    t_w = float(np.median(ts))
    n_solved = grid.n_omega // 2 + 1
    total = t_pairs + t_hist + n_solved * (t_chi + t_w)
    omp = int(os.environ.get("OMP_NUM_THREADS", "0") or 0) or os.cpu_count()
    nblas = blas_threads()
    # context: one W solve with a single BLAS thread (the paper's runs used one core)
    t_w1 = None
    try:
        from threadpoolctl import threadpool_limits

        with threadpool_limits(limits=1):
            t0 = time.perf_counter()
            o.screened_W(mol.v, chi)
            t_w1 = time.perf_counter() - t0
    except ImportError:
        pass
    model = None
    try:
        with open("/proc/cpuinfo") as f:
            model = next((ln.split(":", 1)[1].strip() for ln in f if ln.startswith("model name")), None)
    except OSError:
        pass
    return {
        "value": grid.n_omega / total,
        "unit": "W(omega)/s",
        "solves_per_s": n_solved / total,
        "cores": max(nblas, omp),
        "host_cpus": os.cpu_count(),
        "cpu_model": model,
        "one_thread_W_solve_s": t_w1,
        "kind": "oracle",
        "sample": ("pair vectors in full (%.1fs); int64 histogram (C, %d OpenMP threads) on %d of %d entries "
                   "(scaled); chi0 direct sum at one frequency on the same entries (scaled x%d frequencies); "
                   "LAPACK zgesv W solve (%d BLAS threads) at N=%d on %d frequencies (median %.2fs, scaled x%d); "
                   "the %d solved frequencies of the conjugate mirror, as on the GPU")
                  % (t_pairs, omp, n_samp, n_upper, n_solved, nblas, n, len(ts), t_w, n_solved, n_solved),
    }


def base_record(args, metric, value, unit, t_step, dtype, config, higher=True):
    return {
        "metric": metric,
        "value": value,
        "unit": unit,
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": t_step * 1e3,
        "higher_is_better": higher,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": dtype,
        "data": "synthetic (seeded paper-shaped generators)",
        "config": config,
    }


# kernels whose arithmetic runs on the vector units (FP64 vector peak 78.6 TF)
VALU_KERNELS = {"time_contract", "sigma_contract", "cauchy_add"}
PEAK_BY_CLASS = {"zgemm": PEAK_FP64, "formA": PEAK_FP64, "dzgemm": PEAK_FP64, "zdgemm": PEAK_FP64,
                 "dgemm": PEAK_FP64, "cgemm": PEAK_FP32}


def executed(stats):
    """The library counts a complex product as 8 M N K; the kernels that form it
    from three real products run 6 M N K of them on the matrix cores.  The counts
    that a fraction of the hardware's peak can be taken of."""
    return [dict(s, flops=0.75 * s["flops"]) if s["name"].startswith(("zgemm3m", "block_solve")) else s
            for s in stats]


def kernel_roofline(stats):
    """Dominant kernel (largest summed time) from the library's live per-launch
    HIP event timings: achieved = summed flops (as given: see executed) or bytes
    over the summed launch durations."""
    st = [s for s in stats if s["ms"] > 0]
    if not st:
        return None
    d = max(st, key=lambda s: s["ms"])
    sec = d["ms"] / 1e3
    if d["flops"] > 0 and d["name"] in VALU_KERNELS:
        # FP64 work on the vector units: against the FP64 vector peak
        achieved = d["flops"] / sec / 1e12
        rec = {"bound": "alu", "achieved": achieved, "peak": PEAK_FP64 / 1e12, "unit": "TFLOP/s",
               "frac": achieved / (PEAK_FP64 / 1e12), "flops_per_launch": d["flops"] / d["launches"]}
    elif d["flops"] > 0 and d["name"] != "hist":
        peak = PEAK_BY_CLASS.get(d["name"].split("_")[0], PEAK_FP64) / 1e12
        achieved = d["flops"] / sec / 1e12
        rec = {"bound": "mfma", "achieved": achieved, "peak": peak, "unit": "TFLOP/s", "frac": achieved / peak,
               "flops_per_launch": d["flops"] / d["launches"]}
    else:
        achieved = d["bytes"] / sec / 1e9
        rec = {"bound": "hbm", "achieved": achieved, "peak": 8000.0, "unit": "GB/s", "frac": achieved / 8000.0,
               "bytes_per_launch": d["bytes"] / d["launches"]}
    rec.update({"traffic": stored_traffic() if d["name"] == TRAFFIC_CLASS else None,
                "kernel": d["name"], "launches": d["launches"],
                "avg_launch_us": d["ms"] * 1e3 / d["launches"]})
    rec["all_kernels"] = {s["name"]: {"launches": s["launches"], "ms": round(s["ms"], 3),
                                      "TFLOP/s": round(s["flops"] / (s["ms"] / 1e3) / 1e12, 2) if s["flops"] else None,
                                      "GB/s": round(s["bytes"] / (s["ms"] / 1e3) / 1e9, 1)} for s in st}
    return rec


def live_roofline(ctx):
    return kernel_roofline(executed(ctx.profile_read()))


# ---------------------------------------------------------------------- single molecule
def run_single(args, gw, gs, torch, mol, grid, workload):
    n, N = mol.n_prod, grid.n_omega
    dev = torch.device("cuda:0")
    dm = gw.DeviceMolecule(mol, device=dev)
    g = gw.make_grid(N, grid.omega_min, grid.omega_max, grid.eps)
    ctx = gw.Context(0)
    chi = torch.empty((N, n, n), dtype=torch.complex128, device=dev)
    W = torch.empty((N, n, n), dtype=torch.complex128, device=dev)
    stream = torch.cuda.current_stream()
    forms = [f for f in args.forms.split(",") if f]
    sample_js = [0, N // 2, N // 2 + 30, N // 2 + 100, N - 1, 200]
    W_ref = None
    results, roofs = {}, {}
    for form in forms:
        # "<precision>_A": A = 1 - v chi0 formed from v a0 (gw_build_A), W from A
        route_a = form.endswith("_A")
        base = form[:-2] if route_a else form
        p = FORMS[base]
        # the FP64 forms (the headline candidates) take the requested steps;
        # the refined forms, several times slower on this chip, at most five
        warm, steps = (args.warmup, args.steps) if base == "fp64" else (min(args.warmup, 1), min(args.steps, 5))
        ev, reps = [], []
        for it in range(warm + steps):
            timed = it >= warm
            if timed and base == "fp64":
                ctx.profile_begin()
            torch.cuda.synchronize()
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            e2 = torch.cuda.Event(enable_timing=True)
            t0 = time.perf_counter()
            e0.record(stream)
            if route_a:  # chi holds A
                ctx.build_A(dm.struct, dm.v, g, chi, stream=stream, report=False)
            else:
                ctx.build_chi0(dm.struct, g, chi, stream=stream, report=False)
            e1.record(stream)
            if route_a:
                rep = ctx.solve_W_A(dm.v, n, chi, N, W, prec=p, tol=1e-7, stream=stream, report=True)
            else:
                rep = ctx.solve_W(dm.v, n, chi, N, W, prec=p, tol=1e-7, stream=stream, report=True)
            e2.record(stream)
            torch.cuda.synchronize()
            wall = time.perf_counter() - t0
            if timed:
                ev.append((e0.elapsed_time(e1) / 1e3, e1.elapsed_time(e2) / 1e3, wall))
                reps.append((rep.max_iter, rep.n_fallback, rep.max_rel_update))
            log("%s step %d: chi0 %.3fs solve %.3fs wall %.3fs iters %d fallback %d" % (
                form, it, e0.elapsed_time(e1) / 1e3, e1.elapsed_time(e2) / 1e3, wall, rep.max_iter,
                rep.n_fallback))
        if base == "fp64":
            roofs[form] = live_roofline(ctx)
            ctx.profile_end()
        samp = W[sample_js].cpu().numpy()
        if form == "fp64":
            W_ref = samp
            err = 0.0
        else:
            err = None if W_ref is None else float(max(
                np.linalg.norm(samp[i] - W_ref[i]) / np.linalg.norm(W_ref[i]) for i in range(len(sample_js))))
        walls = np.array([e[2] for e in ev])
        results[form] = {
            "t_chi0": float(np.median([e[0] for e in ev])),
            "t_solve": float(np.median([e[1] for e in ev])),
            "t_step": float(np.median(walls)),
            "p50_ms": float(np.percentile(walls, 50) * 1e3),
            "p99_ms": float(np.percentile(walls, 99) * 1e3),
            "n_solved": int(rep.n_solved),
            "max_iter": int(max(r[0] for r in reps)),
            "fallback": int(max(r[1] for r in reps)),
            "rel_err_vs_fp64": err,
            "route_a": route_a,
            "steps": steps,
        }
    ok = {f: r for f, r in results.items() if r["rel_err_vs_fp64"] is None or r["rel_err_vs_fp64"] <= 1e-6}
    best = min(ok, key=lambda f: ok[f]["t_step"])
    r = results[best]
    out = base_record(
        args, "W(omega) freq-solves/sec at N_prod=2000 (mixed vs FP64, same GPU); p50/p99 latency",
        N / r["t_step"], "W(omega)/s", r["t_step"], "f64" if best.startswith("fp64") else "f32+f64",
        {"workload": workload, "n_prod": n, "n_omega": N, "n_pairs": mol.n_pairs, "form": best,
         "parallelism": "none (1 GPU)"})
    out["forms"] = {}
    for f, v in results.items():
        ach, pk = solve_roofline(n, v["n_solved"], v["t_solve"], v["max_iter"], not f.startswith("fp64"),
                                 form_a=not v["route_a"])
        out["forms"][f] = {"W_per_s": N / v["t_step"], "solves_per_s": v["n_solved"] / v["t_step"],
                           "t_chi0_s": v["t_chi0"], "t_solve_s": v["t_solve"], "p50_ms": v["p50_ms"],
                           "p99_ms": v["p99_ms"], "max_ir_steps": v["max_iter"], "fp64_fallbacks": v["fallback"],
                           "rel_err_vs_fp64": v["rel_err_vs_fp64"], "steps_timed": v["steps"],
                           "solve_TFLOPs": ach, "solve_roofline_frac": ach / pk}
    out["step_latency_ms"] = {"p50": r["p50_ms"], "p99": r["p99_ms"]}
    if roofs:
        # the headline form's kernels when they were timed, else the FP64 chi0 route's
        out["roofline"] = roofs.get(best, roofs.get("fp64", next(iter(roofs.values()))))
    out["step_roofline"] = step_roofline(n, N, r["n_solved"], rep_nhb(gw, mol, grid), r["t_step"], r["max_iter"],
                                         not best.startswith("fp64"), r["route_a"])
    ctx.close()
    del chi, W, dm
    torch.cuda.empty_cache()
    if not args.no_serving and workload.startswith("chain40_nprod2000"):
        # the serving form of the path (gw_submit .. gw_poll) on a bounded
        # window of the Poisson workload, so that p50/p99 come from this run
        legs = serving_legs(args, gw, gs, torch, pool_size=args.serve_pool, duration=args.serve_duration)
        out["serving"] = legs
        o = legs["overloaded"]
        out["latency_ms"] = {"p50": o["p50_ms"], "p99": o["p99_ms"],
                             "below_capacity_p50": legs["below_capacity"]["p50_ms"],
                             "below_capacity_p99": legs["below_capacity"]["p99_ms"],
                             "definition": "gw_submit to gw_poll completion over every arrival; requests still "
                                           "queued at the end of the arrival window are cancelled and counted at "
                                           "their age then (a lower bound)"}
    if not args.no_cpu_baseline:
        log("timing the oracle on the host")
        out["cpu_baseline"] = cpu_baseline(mol, grid)
    return out


def rep_nhb(gw, mol, grid):
    g = gw.make_grid(grid.n_omega, grid.omega_min, grid.omega_max, grid.eps)
    return gw.query_sizes(mol.n_orb, mol.n_occ, mol.n_prod, np.ascontiguousarray(mol.eig), g).n_hbins


def step_roofline(n, N, n_solved, nhb, t_step, n_ir, mixed, route_a):
    """Whole-step roofline of the headline form: the algorithmic matrix-core
    work of one step (the solve's products per solved frequency, plus on the A
    route the n_hbins - 1 real products v a0 of 2 N^3 each) at the FP64 and
    FP32 matrix peaks, over the measured step time.  The histogram, the FFT
    and the copies are not counted in the numerator, so the fraction is a
    lower bound on how close the step is to its matrix-core roofline."""
    fl = solve_flops(n, n_solved, n_ir, mixed, form_a=not route_a)
    fp64 = fl["fp64"] + (2.0 * float(n) ** 3 * (nhb - 1) if route_a else 0.0)
    fp32 = fl["fp32"]
    t_roof = fp64 / PEAK_FP64 + fp32 / PEAK_FP32
    return {"bound": "mfma", "flops_fp64": fp64, "flops_fp32": fp32, "t_roof_s": t_roof, "t_step_s": t_step,
            "achieved_TFLOPs": (fp64 + fp32) / t_step / 1e12, "frac": t_roof / t_step}


# ---------------------------------------------------------------------- compressed cluster
def run_c2(args, gw, gs, torch):
    log("generating the 120-atom cluster")
    mol = gs.make_config(2)
    grid = gs.config_grid(2)
    k = 1500
    n, N = mol.n_prod, grid.n_omega
    dev = torch.device("cuda:0")
    dm = gw.DeviceMolecule(mol, device=dev)
    g = gw.make_grid(N, grid.omega_min, grid.omega_max, grid.eps)
    ctx = gw.Context(0, budget_bytes=96 << 30)
    Q = torch.empty((n, k), dtype=torch.float64, device=dev)
    S = torch.empty((k, k), dtype=torch.float64, device=dev)
    chi = torch.empty((N, k, k), dtype=torch.complex128, device=dev)
    X = torch.empty((N, k, k), dtype=torch.complex128, device=dev)
    stream = torch.cuda.current_stream()
    forms = [f for f in args.forms.split(",") if f]
    sample_js = [0, N // 2, N // 2 + 60, N // 2 + 200, N - 1, 400]
    res, X_ref = {}, None
    for form in forms:
        # "<precision>_A": A = 1 - S chi_hat formed from S a0_hat (gw_build_A_compressed), X from A
        route_a = form.endswith("_A")
        base = form[:-2] if route_a else form
        ts = []
        for it in range(args.warmup + args.steps):
            torch.cuda.synchronize()
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
            t0 = time.perf_counter()
            ev[0].record(stream)
            ctx.compress_basis(dm.v, n, k, Q, S, stream=stream)
            ev[1].record(stream)
            if route_a:  # chi holds A
                ctx.build_A_compressed(dm.struct, S, Q, k, g, chi, stream=stream, report=False)
            else:
                ctx.build_chi0(dm.struct, g, chi, basis=Q, k=k, stream=stream, report=False)
            ev[2].record(stream)
            if route_a:
                rep = ctx.solve_W_A(S, k, chi, N, X, prec=FORMS[base], tol=1e-7, stream=stream)
            else:
                rep = ctx.solve_W(S, k, chi, N, X, prec=FORMS[base], tol=1e-7, stream=stream)
            ev[3].record(stream)
            torch.cuda.synchronize()
            wall = time.perf_counter() - t0
            parts = [ev[i].elapsed_time(ev[i + 1]) / 1e3 for i in range(3)]
            log("c2 %s step %d: basis %.3fs chi_hat %.3fs solve %.3fs wall %.3fs iters %d fallback %d" % (
                form, it, *parts, wall, rep.max_iter, rep.n_fallback))
            if it >= args.warmup:
                ts.append((wall, *parts, rep.max_iter, rep.n_fallback))
        samp = X[sample_js].cpu().numpy()
        if X_ref is None:
            X_ref = samp
        err = float(max(np.linalg.norm(samp[i] - X_ref[i]) / np.linalg.norm(X_ref[i])
                        for i in range(len(sample_js))))
        a = np.array(ts)
        res[form] = {"t_step": float(np.median(a[:, 0])), "t_basis": float(np.median(a[:, 1])),
                     "t_chi_hat": float(np.median(a[:, 2])), "t_solve": float(np.median(a[:, 3])),
                     "max_iter": int(a[:, 4].max()), "fallback": int(a[:, 5].max()),
                     "rel_err_vs_first_form": err}
    ok = {f: r for f, r in res.items() if r["rel_err_vs_first_form"] <= 1e-6}
    best = min(ok, key=lambda f: ok[f]["t_step"])
    r = res[best]
    out = base_record(args, "W(omega)/s, 120-atom cluster, top-1500 compressed, 2048 points", N / r["t_step"],
                      "W(omega)/s", r["t_step"], "f64" if best.startswith("fp64") else "f32+f64",
                      {"workload": "cluster120_k1500_nomega2048", "n_prod": n, "k": k, "n_omega": N,
                       "n_pairs": mol.n_pairs, "form": best, "parallelism": "none (1 GPU)"})
    out["forms"] = {}
    for f, v in res.items():
        ach, pk = solve_roofline(k, N // 2 + 1, v["t_solve"], v["max_iter"], not f.startswith("fp64"),
                                 form_a=not f.endswith("_A"))
        out["forms"][f] = dict(v, W_per_s=N / v["t_step"], solve_TFLOPs=ach, solve_roofline_frac=ach / pk)
    ctx.close()
    return out


# ---------------------------------------------------------------------- paper's subspace
def run_c2pair(args, gw, gs, torch):
    """120-atom cluster compressed to the paper's own subspace (Section 7.A):
    pairs with F - E < 0.4 Ha generate it, k = 256 of its dimensions kept;
    one step = basis + chi_hat + X(omega) on all 2048 points."""
    log("generating the 120-atom cluster")
    mol = gs.make_config(2)
    grid = gs.config_grid(2)
    k, thr = 256, 0.4
    n, N = mol.n_prod, grid.n_omega
    dev = torch.device("cuda:0")
    dm = gw.DeviceMolecule(mol, device=dev)
    g = gw.make_grid(N, grid.omega_min, grid.omega_max, grid.eps)
    ctx = gw.Context(0, budget_bytes=96 << 30)
    Z = torch.empty((n, k), dtype=torch.float64, device=dev)
    U = torch.empty_like(Z)
    R = torch.empty((n, n), dtype=torch.float64, device=dev)
    ones = torch.ones(k, dtype=torch.float64, device=dev)
    chi = torch.empty((N, k, k), dtype=torch.complex128, device=dev)
    X = torch.empty_like(chi)
    stream = torch.cuda.current_stream()
    ts = []
    for it in range(args.warmup + args.steps):
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        t0 = time.perf_counter()
        ev[0].record(stream)
        nr = ctx.pair_basis(dm.struct, dm.v, thr, k, Z, U, R, stream=stream)
        ev[1].record(stream)
        ctx.build_chi0(dm.struct, g, chi, basis=U, k=k, stream=stream, report=False)
        ev[2].record(stream)
        ctx.solve_W(ones, k, chi, N, X, v_is_diag=True, stream=stream, report=False)
        ev[3].record(stream)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        parts = [ev[i].elapsed_time(ev[i + 1]) / 1e3 for i in range(3)]
        log("c2pair step %d: basis %.3fs chi_hat %.3fs solve %.3fs wall %.3fs (N_rank %d)" % (it, *parts, wall, nr))
        if it >= args.warmup:
            ts.append((wall, *parts))
    a = np.median(np.array(ts), axis=0)
    out = base_record(args, "W(omega)/s, 120-atom cluster in the paper's pair subspace (k=256), 2048 points",
                      N / a[0], "W(omega)/s", a[0], "f64",
                      {"workload": "cluster120_pairbasis_thr0.4_k256_nomega2048", "n_prod": n, "k": k,
                       "n_rank": nr, "e_threshold_Ha": thr, "n_omega": N, "parallelism": "none (1 GPU)"})
    out["phases_s"] = {"basis": a[1], "chi_hat": a[2], "solve": a[3]}
    ctx.close()
    return out


# ---------------------------------------------------------------------- two windows
def run_two_window(args, gw, gs, torch):
    """The 2000-product molecule with two spectral windows (Section 5.B): a
    fine 256-point mesh over |omega| < 0.5 Ha and a coarse 256-point mesh over
    |omega| < 4 Ha, eps = 1.5 domega in each.  One step = gw_build_chi0_2w
    (both meshes) + W on both meshes (in place, 2 x 129 factorised points)."""
    log("generating molecule")
    mol = gs.truncate_products(gs.make_config(1), N_PROD)
    small, large = gs.two_window_grids()
    n = mol.n_prod
    dev = torch.device("cuda:0")
    dm = gw.DeviceMolecule(mol, device=dev)
    gsm = gw.make_grid(small.n_omega, small.omega_min, small.omega_max, small.eps)
    glg = gw.make_grid(large.n_omega, large.omega_min, large.omega_max, large.eps)
    ctx = gw.Context(0)
    cs = torch.empty((small.n_omega, n, n), dtype=torch.complex128, device=dev)
    cl = torch.empty((large.n_omega, n, n), dtype=torch.complex128, device=dev)
    stream = torch.cuda.current_stream()
    ts = []
    roof = None
    for it in range(args.warmup + args.steps):
        timed = it >= args.warmup
        if timed and roof is None:
            ctx.profile_begin()
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        t0 = time.perf_counter()
        ev[0].record(stream)
        ctx.build_chi0_2w(dm.struct, gsm, glg, cs, cl, stream=stream, report=False)
        ev[1].record(stream)
        ctx.solve_W(dm.v, n, cs, small.n_omega, cs, stream=stream, report=False)
        ev[2].record(stream)
        ctx.solve_W(dm.v, n, cl, large.n_omega, cl, stream=stream, report=False)
        ev[3].record(stream)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        parts = [ev[i].elapsed_time(ev[i + 1]) / 1e3 for i in range(3)]
        log("two-window step %d: chi0 both meshes %.3fs W fine %.3fs W coarse %.3fs wall %.3fs" % (it, *parts,
                                                                                                    wall))
        if timed:
            ts.append((wall, *parts))
            if roof is None:
                roof = live_roofline(ctx)
                ctx.profile_end()
    a = np.median(np.array(ts), axis=0)
    n_pts = small.n_omega + large.n_omega
    out = base_record(args, "W(omega)/s, 2000 products, two spectral windows (256 fine + 256 coarse points)",
                      n_pts / a[0], "W(omega)/s", a[0], "f64",
                      {"workload": "chain40_nprod2000_two_windows_256x0.5Ha_256x4Ha", "n_prod": n,
                       "n_omega_small": small.n_omega, "omega_max_small_Ha": small.omega_max,
                       "n_omega_large": large.n_omega, "omega_max_large_Ha": large.omega_max,
                       "parallelism": "none (1 GPU)"})
    out["phases_s"] = {"chi0_both_meshes": a[1], "W_fine": a[2], "W_coarse": a[3]}
    out["roofline"] = roof
    ctx.close()
    return out


# ---------------------------------------------------------------------- the paper's a0 route
def run_time_route(args, gw, gs, torch):
    """The 2000-product molecule on the 1024-point mesh with a0 built by the
    paper's own route (Section 8.A: densities to time, local product per
    time, back).  One step = gw_build_A_time (a0 by the time route, then A =
    1 - v chi0 from v a0) + W from A on all points (FP64).  The pair-route
    build of A is timed beside it for comparison."""
    log("generating molecule")
    mol = gs.truncate_products(gs.make_config(1), N_PROD)
    grid = gs.config_grid(1)
    n, N = mol.n_prod, grid.n_omega
    dev = torch.device("cuda:0")
    dm = gw.DeviceMolecule(mol, device=dev)
    g = gw.make_grid(N, grid.omega_min, grid.omega_max, grid.eps)
    ctx = gw.Context(0)
    chi = torch.empty((N, n, n), dtype=torch.complex128, device=dev)
    W = torch.empty_like(chi)
    stream = torch.cuda.current_stream()
    ts, roof = [], None
    for it in range(args.warmup + args.steps):
        timed = it >= args.warmup
        if timed and roof is None:
            ctx.profile_begin()
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        t0 = time.perf_counter()
        ev[0].record(stream)
        ctx.build_A_time(dm.struct, dm.v, g, chi, stream=stream, report=False)  # chi holds A
        ev[1].record(stream)
        ctx.solve_W_A(dm.v, n, chi, N, W, stream=stream, report=False)
        ev[2].record(stream)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        parts = [ev[0].elapsed_time(ev[1]) / 1e3, ev[1].elapsed_time(ev[2]) / 1e3]
        if timed and roof is None:
            roof = live_roofline(ctx)
            ctx.profile_end()
        # the pair-route build of the same A, outside the step, for comparison
        ev[3].record(stream)
        ctx.build_A(dm.struct, dm.v, g, chi, stream=stream, report=False)
        e5 = torch.cuda.Event(enable_timing=True)
        e5.record(stream)
        torch.cuda.synchronize()
        t_pair = ev[3].elapsed_time(e5) / 1e3
        log("time-route step %d: A (time route) %.3fs solve %.3fs wall %.3fs | A (pair route) %.3fs" % (
            it, parts[0], parts[1], wall, t_pair))
        if timed:
            ts.append((wall, parts[0], parts[1], t_pair))
    a = np.median(np.array(ts), axis=0)
    out = base_record(args, "W(omega)/s, 2000 products, 1024 points, a0 by the paper's time-domain route",
                      N / a[0], "W(omega)/s", a[0], "f64",
                      {"workload": "chain40_nprod2000_nomega1024_time_route", "n_prod": n, "n_omega": N,
                       "n_orb": mol.n_orb, "parallelism": "none (1 GPU)"})
    out["phases_s"] = {"A_time_route": a[1], "solve": a[2], "A_pair_route": a[3]}
    out["roofline"] = roof
    ctx.close()
    return out


# ---------------------------------------------------------------------- self-energy
def run_self_energy(args, gw, gs, torch):
    """The 2000-product molecule on the 1024-point mesh carried through to the
    GW self-energy: one step = A = 1 - v chi0 from v a0 + W (FP64, all points;
    the headline route) + sigma+- by the
    time-by-time convolution + Sigma on all points + exchange + Dyson's
    equation and the DOS on all points (V_xc = 0: the synthetic orbitals carry
    no DFT potential; the arithmetic is the same).  value = Sigma(omega)
    points per second for the whole step."""
    log("generating molecule")
    mol = gs.truncate_products(gs.make_config(1), N_PROD)
    grid = gs.config_grid(1)
    n, N, no = mol.n_prod, grid.n_omega, mol.n_orb
    dev = torch.device("cuda:0")
    dm = gw.DeviceMolecule(mol, device=dev)
    g = gw.make_grid(N, grid.omega_min, grid.omega_max, grid.eps)
    ctx = gw.Context(0)
    chi = torch.empty((N, n, n), dtype=torch.complex128, device=dev)
    W = torch.empty_like(chi)
    S = torch.empty((N, no, no), dtype=torch.complex128, device=dev)
    Sx = torch.empty((no, no), dtype=torch.float64, device=dev)
    dos = torch.empty((N,), dtype=torch.float64, device=dev)
    stream = torch.cuda.current_stream()
    ts, roof = [], None
    for it in range(args.warmup + args.steps):
        timed = it >= args.warmup
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(5)]
        t0 = time.perf_counter()
        ev[0].record(stream)
        ctx.build_A(dm.struct, dm.v, g, chi, stream=stream, report=False)  # chi holds A
        ev[1].record(stream)
        ctx.solve_W_A(dm.v, n, chi, N, W, stream=stream, report=False)
        ev[2].record(stream)
        if timed and roof is None:
            ctx.profile_begin()
        ctx.self_energy(dm.struct, g, W, S, v=dm.v, Sigma_x_out=Sx, stream=stream, report=False)
        ev[3].record(stream)
        ctx.dyson_dos(dm.struct, g, dos, Sigma_c=S, Sigma_x=Sx, stream=stream, report=False)
        ev[4].record(stream)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        parts = [ev[i].elapsed_time(ev[i + 1]) / 1e3 for i in range(4)]
        if timed and roof is None:
            roof = live_roofline(ctx)
            ctx.profile_end()
        log("self-energy step %d: A %.3fs W %.3fs Sigma %.3fs Dyson+DOS %.3fs wall %.3fs" % (it, *parts, wall))
        if timed:
            ts.append((wall, *parts))
    a = np.median(np.array(ts), axis=0)
    out = base_record(args, "Sigma(omega)/s, 2000 products, 1024 points (A = 1 - v chi0, W, sigma by time-domain convolution, "
                            "Sigma, exchange, Dyson + DOS)", N / a[0], "Sigma(omega)/s", a[0], "f64",
                      {"workload": "chain40_nprod2000_nomega1024_self_energy", "n_prod": n, "n_orb": no,
                       "n_omega": N, "parallelism": "none (1 GPU)"})
    out["phases_s"] = {"A_from_v_a0": a[1], "W": a[2], "self_energy": a[3], "dyson_dos": a[4]}
    out["roofline_sigma_dyson_phases"] = roof
    ctx.close()
    return out


# ---------------------------------------------------------------------- batched
def run_c3(args, gw, gs, torch):
    grid = gs.config_grid(3)
    N = grid.n_omega
    log("generating %d chain molecules" % args.mols)
    mols = gs.batch_molecules(args.mols)
    dev = torch.device("cuda:0")
    g = gw.make_grid(N, grid.omega_min, grid.omega_max, grid.eps)
    ws_budget = 64 << 30
    ctx = gw.Context(0, budget_bytes=ws_budget)
    stream = torch.cuda.current_stream()

    def next_group(start):
        # consecutive molecules whose in-place outputs fit in what is free now,
        # leaving room for the context's (grow-only) workspaces (the in-place
        # molecules' v a0 bins take up to 18 GB of them)
        torch.cuda.empty_cache()
        free, _ = torch.cuda.mem_get_info()
        cap = free - (88 << 30)
        grp, used = [], 0
        for i in range(start, len(mols)):
            b = N * mols[i].n_prod ** 2 * 16
            if grp and used + b > cap:
                break
            grp.append(i)
            used += b
        return grp

    forms = [f for f in args.forms.split(",") if f]
    res = {}
    for form in forms:
        t_create = t_run = 0.0
        solves = 0
        flops = 0.0
        worst_fb = 0
        start, gi, n_groups = 0, 0, 0
        rec = {"mode": None, "steps": 0, "launches": 0, "products": 0}
        while start < len(mols):
            grp = next_group(start)
            start = grp[-1] + 1
            n_groups += 1
            dms = [gw.DeviceMolecule(mols[i], device=dev) for i in grp]
            bufs = [torch.empty((N, mols[i].n_prod, mols[i].n_prod), dtype=torch.complex128, device=dev)
                    for i in grp]
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            b = ctx.batch_create([d.struct for d in dms], [d.v for d in dms], g, bufs, bufs, prec=FORMS[form],
                                 tol=1e-6, n_refine=2, stream=stream)
            torch.cuda.synchronize()
            tc = time.perf_counter() - t0
            st = b.stats()
            rec["mode"] = {0: "molecules on parallel branches", 1: "lock steps (aligned at the end)",
                           2: "lock steps (aligned at the start)"}[st["mode"]]
            for k in ("steps", "launches", "products"):
                rec[k] += st[k]
            t0 = time.perf_counter()
            reps = b.run(stream=stream)
            torch.cuda.synchronize()
            tr = time.perf_counter() - t0
            t_create += tc
            t_run += tr
            solves += sum(r.n_solved for r in reps)
            worst_fb = max(worst_fb, max(r.n_fallback for r in reps))
            for i in grp:
                # in place: A is formed from v a0 (no 4N^3 product per frequency)
                fl = solve_flops(mols[i].n_prod, N // 2 + 1, 2, form != "fp64", form_a=False)
                flops += fl["fp64"] + fl["fp32"]
            log("c3 %s group %d: %d molecules (n_prod %d..%d) create %.2fs replay %.2fs" % (
                form, gi, len(grp), min(mols[i].n_prod for i in grp), max(mols[i].n_prod for i in grp), tc, tr))
            b.close()
            del bufs, dms
            gi += 1
        res[form] = {"t_replay_s": t_run, "t_create_s": t_create, "W_per_s": len(mols) * N / t_run,
                     "solves_per_s": solves / t_run, "W_per_s_incl_create": len(mols) * N / (t_run + t_create),
                     "solve_TFLOPs": flops / t_run / 1e12, "fp64_fallbacks": worst_fb, "groups": n_groups,
                     "recording": rec}
    best = max(res, key=lambda f: res[f]["W_per_s"])
    r = res[best]
    out = base_record(args, "W(omega)/s, %d chain molecules batched (solves in lock steps) in recorded hipGraphs, "
                            "512 points" % len(mols),
                      r["W_per_s"], "W(omega)/s", r["t_replay_s"], "f64" if best == "fp64" else "f32+f64",
                      {"workload": "batch%d_chains_8to80_nomega512" % len(mols), "molecules": len(mols),
                       "n_prod_min": min(m.n_prod for m in mols), "n_prod_max": max(m.n_prod for m in mols),
                       "n_omega": N, "form": best, "in_place": True, "parallelism": "none (1 GPU)"})
    out["forms"] = res
    ctx.close()
    return out


# ---------------------------------------------------------------------- serving
def serving_pool(gs, gw, torch, n_pool, lo=10, hi=200):
    """Cluster molecules at n_pool atom counts spaced evenly in log between lo
    and hi (the midpoints of n_pool equal-probability slices of the
    log-uniform arrival distribution).  Generating every arrival's own cluster
    would take about a second each on the host, so each arrival is served the
    molecule whose atom count is nearest to its own drawn count; the record
    reports how far that moves the sizes and the cost."""
    la, lb = math.log(lo), math.log(hi)
    counts = sorted(set(int(round(math.exp(la + (k + 0.5) * (lb - la) / n_pool))) for k in range(n_pool)))
    dev = torch.device("cuda:0")
    pool = []
    for c in counts:
        m = gs.serving_molecule(c, c)
        pool.append((c, m, gw.DeviceMolecule(m, device=dev)))
    return pool


def _nearest(pool, c):
    return min(range(len(pool)), key=lambda i: (abs(math.log(pool[i][0] / c)), pool[i][0]))


def serve_leg(gw, g, N, pool, rate, duration, seed, prec, cancel_at_end):
    """One Poisson window: submit each arrival on time, poll, release.
    Latency = gw_submit .. gw_poll completion.  With cancel_at_end, requests
    still queued when the window closes are cancelled and counted at their age
    then (censored: a lower bound on their latency)."""
    times, counts = arrival_stream(rate, duration, seed)
    picks = [_nearest(pool, int(c)) for c in counts]
    ctx = gw.Context(0)
    pending = {}
    lat, cens = [], []
    done = cancelled = delivered = 0
    i = 0
    t_start = time.perf_counter()
    while True:
        now = time.perf_counter() - t_start
        while i < len(times) and times[i] <= now:
            _, m, dm = pool[picks[i]]
            k = min(m.n_prod, 1500)
            t = ctx.submit(dm.struct, dm.v, g, k_compress=k, prec=prec, tol=1e-7)
            pending[t] = times[i]
            i += 1
        for t in list(pending):
            r = ctx.poll(t)
            if r is not None:
                lat.append(time.perf_counter() - t_start - pending.pop(t))
                ctx.release(t)
                done += 1
                delivered += N
        if i >= len(times):
            break
        time.sleep(0.001)
    t_window = time.perf_counter() - t_start
    if cancel_at_end:
        for t in list(pending):
            try:
                ctx.release(t)
            except gw.GwError:
                continue  # running: it will complete below
            cens.append(t_window - pending.pop(t))
            cancelled += 1
    while pending:
        for t in list(pending):
            r = ctx.poll(t)
            if r is not None:
                lat.append(time.perf_counter() - t_start - pending.pop(t))
                ctx.release(t)
                done += 1
                delivered += N
        time.sleep(0.002)
    wall = time.perf_counter() - t_start
    ctx.close()
    every = np.array(lat + cens) * 1e3
    lat_ms = np.array(lat) * 1e3
    served = np.array([pool[p][1].n_prod for p in picks], dtype=float)
    # size fidelity: the arrivals' own drawn atom counts against the served ones
    drawn_atoms = np.asarray(counts, dtype=float)
    served_atoms = np.array([pool[p][0] for p in picks], dtype=float)
    return {
        "offered_per_s": rate, "window_s": duration, "arrivals": len(times), "completed": done,
        "cancelled": cancelled, "completed_fraction": done / max(1, len(times)),
        "sustained_requests_per_s": done / wall, "sustained_W_per_s": delivered / wall, "wall_s": wall,
        "p50_ms": float(np.percentile(every, 50)) if len(every) else None,
        "p99_ms": float(np.percentile(every, 99)) if len(every) else None,
        "completed_p50_ms": float(np.percentile(lat_ms, 50)) if done else None,
        "completed_p99_ms": float(np.percentile(lat_ms, 99)) if done else None,
        "censored_at_window_end": cancelled,
        "size_fidelity": {
            "pool_atom_counts": [c for c, _, _ in pool],
            "mean_abs_rel_atom_error": float(np.mean(np.abs(served_atoms / drawn_atoms - 1.0))) if len(picks) else None,
            "mean_n_prod_served": float(served.mean()) if len(picks) else None,
            "cost_ratio_served_vs_drawn": float(np.mean(np.minimum(served_atoms * 60.0, 1500.0) ** 3) /
                                                np.mean(np.minimum(drawn_atoms * 60.0, 1500.0) ** 3))
            if len(picks) else None,
        },
    }


def arrival_stream(rate, duration, seed):
    sys.path.insert(0, HERE)
    import gw_synth as gs

    return gs.serving_stream(rate=rate, duration=duration, seed=seed)


def serving_legs(args, gw, gs, torch, pool_size, duration):
    grid = gs.config_grid(4)
    N = grid.n_omega
    g = gw.make_grid(N, grid.omega_min, grid.omega_max, grid.eps)
    log("serving: generating a pool of %d cluster molecules" % pool_size)
    pool = serving_pool(gs, gw, torch, pool_size)
    prec = 0
    out = {}
    for label, rate, seed, cancel in (("overloaded", args.rate, 4, True), ("below_capacity", args.low_rate, 5, False)):
        out[label] = serve_leg(gw, g, N, pool, rate, duration, seed, prec, cancel)
        log("serving %s: %s" % (label, json.dumps({k: v for k, v in out[label].items() if k != "size_fidelity"})))
    out["form"] = "fp64, k = min(N_prod, 1500) top-k compression, 1024 points"
    return out


def run_c4(args, gw, gs, torch):
    grid = gs.config_grid(4)
    N = grid.n_omega
    legs = serving_legs(args, gw, gs, torch, pool_size=args.pool, duration=args.duration)
    o = legs["overloaded"]
    rec = base_record(args, "served W(omega)/s (sustained) with p50/p99 latency, Poisson arrivals",
                      o["sustained_W_per_s"], "W(omega)/s", o["wall_s"], "f64",
                      {"workload": "serve_poisson%g_clusters10to200_k1500_nomega1024" % args.rate,
                       "duration_s": args.duration, "pool": args.pool, "n_omega": N, "parallelism": "none (1 GPU)"})
    rec["latency_ms"] = {"p50": o["p50_ms"], "p99": o["p99_ms"]}
    rec["serving"] = legs
    return rec


# ---------------------------------------------------------------------- profiles
# Kernel whose HBM traffic the roofline reports, and the source it is built from.
TRAFFIC_KERNEL = "k_zgemm<4, 2, 2, true, true>"
TRAFFIC_CLASS = "zgemm3m_128x64"  # the same kernel in the library's live timing
TRAFFIC_FILE = os.path.join(HERE, "profiles", "hbm_traffic.json")
COPY_BYTES = 1 << 30


def kernel_source_hash():
    """Hash of the sources that define the dominant kernel (the GEMM) and the
    shapes it is launched with (the blocked LU and solves)."""
    import hashlib

    h = hashlib.sha256()
    for name in ("k_gemm.hip", "k_lu.hip"):
        with open(os.path.join(HERE, "paper_1101_2065_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def stored_traffic():
    """HBM bytes per launch of the dominant kernel from the committed counter
    summary, or None when the kernel source changed since it was measured."""
    try:
        with open(TRAFFIC_FILE) as f:
            t = json.load(f)
    except (OSError, ValueError):
        return None
    if t.get("kernel_source_sha256_16") != kernel_source_hash() or t.get("kernel") != TRAFFIC_KERNEL:
        return None
    return t.get("bytes_per_launch")


def _csv_rows(path):
    import csv

    with open(path, newline="") as f:
        return list(csv.DictReader(f))


def summarize_profiles(stats_csv, fetch_csv, write_csv, out_json):
    """Per-kernel HBM traffic from two counter runs (FETCH_SIZE, WRITE_SIZE,
    KiB per dispatch), scaled by the same counters on a plain device copy of
    COPY_BYTES bytes."""
    def per_kernel(path, counter):
        acc = {}
        for r in _csv_rows(path):
            if r.get("Counter_Name") != counter:
                continue
            k = r["Kernel_Name"]
            a = acc.setdefault(k, [0.0, 0])
            a[0] += float(r["Counter_Value"])
            a[1] += 1
        return {k: v[0] / v[1] for k, v in acc.items()}

    fetch = per_kernel(fetch_csv, "FETCH_SIZE")
    write = per_kernel(write_csv, "WRITE_SIZE")
    copy = [k for k in fetch if "MulFunctor" in k]
    copy_k = copy[0] if copy else None
    f_scale = (COPY_BYTES / 1024.0) / fetch[copy_k] if copy_k else 1.0
    w_scale = (COPY_BYTES / 1024.0) / write[copy_k] if copy_k and write.get(copy_k) else 1.0
    rows = []
    for k in sorted(fetch, key=lambda k: -fetch[k]):
        rows.append({"kernel": k, "fetch_KiB": fetch[k], "write_KiB": write.get(k),
                     "bytes": (fetch[k] * f_scale + (write.get(k) or 0.0) * w_scale) * 1024.0})
    dom = [r for r in rows if TRAFFIC_KERNEL in r["kernel"]]
    out = {"kernel": TRAFFIC_KERNEL, "kernel_source_sha256_16": kernel_source_hash(),
           "copy_kernel": copy_k, "fetch_scale": f_scale, "write_scale": w_scale,
           "bytes_per_launch": dom[0]["bytes"] if dom else None, "kernels": rows[:20]}
    with open(out_json, "w") as f:
        json.dump(out, f, indent=1)
    md = [
        "# HBM traffic per dispatch: %s, 40-atom chain truncated to N_prod=2000, "
        "1024 frequencies" % PROFILE_STEP, "",
        "Commands (repository root, one MI355X; one counter per run; OUT is any output directory):", "", "```",
        "rocprofv3 --pmc FETCH_SIZE -d $OUT/pmc_fetch -o run --output-format csv -- python3 bench.py "
        "--forms %s --steps 1 --warmup 0 --no-cpu-baseline --no-serving --copy-calibration" % PROFILE_FORM,
        "rocprofv3 --pmc WRITE_SIZE -d $OUT/pmc_write -o run --output-format csv -- python3 bench.py "
        "--forms %s --steps 1 --warmup 0 --no-cpu-baseline --no-serving --copy-calibration" % PROFILE_FORM,
        "python bench.py --summarize-counters $OUT/prof_n2000/run_kernel_stats.csv "
        "$OUT/pmc_fetch/run_counter_collection.csv $OUT/pmc_write/run_counter_collection.csv",
        "```", "",
        "Calibration: a plain elementwise pass over %d bytes (`%s`) reads FETCH_SIZE %.0f KiB and writes WRITE_SIZE "
        "%.0f KiB per dispatch; factors %.4f (fetch) and %.4f (write) convert the counters to bytes."
        % (COPY_BYTES, (copy_k or "none")[:60], fetch.get(copy_k, 0.0), write.get(copy_k, 0.0), f_scale, w_scale),
        "", "| kernel | dispatches avg FETCH_SIZE KiB | avg WRITE_SIZE KiB | HBM bytes per dispatch |", "|---|---:|---:|---:|"]
    for r in rows[:14]:
        md.append("| `%s` | %.0f | %s | %.3e |" % (r["kernel"][:90], r["fetch_KiB"],
                                                  "%.0f" % r["write_KiB"] if r["write_KiB"] is not None else "-",
                                                  r["bytes"]))
    with open(os.path.join(os.path.dirname(out_json), "hbm_traffic_chain40_n2000.md"), "w") as f:
        f.write("\n".join(md) + "\n")
    print(json.dumps({"copy_kernel": copy_k, "fetch_scale": f_scale, "write_scale": w_scale,
                      "dominant_bytes_per_launch": out["bytes_per_launch"]}))


def summarize_mfma(counter_csv, out_md):
    """Per-kernel matrix-core figures from one rocprofv3 --pmc MfmaUtil
    MfmaFlopsF64 run of the FP64 step: average MFMA busy percentage (busy
    cycles over active cycles of all SIMDs) and executed FP64 matrix flops
    per dispatch (padded tiles included)."""
    acc = {}
    for r in _csv_rows(counter_csv):
        k, c = r["Kernel_Name"], r.get("Counter_Name")
        if c not in ("MfmaUtil", "MfmaFlopsF64"):
            continue
        a = acc.setdefault(k, {"MfmaUtil": [0.0, 0], "MfmaFlopsF64": [0.0, 0]})
        a[c][0] += float(r["Counter_Value"])
        a[c][1] += 1
    rows = []
    for k, a in acc.items():
        fl = a["MfmaFlopsF64"][0] / max(a["MfmaFlopsF64"][1], 1)
        if fl <= 0:
            continue
        rows.append((k, a["MfmaUtil"][1], a["MfmaUtil"][0] / max(a["MfmaUtil"][1], 1), fl))
    rows.sort(key=lambda x: -x[3] * x[1])
    md = ["# Matrix-core use per dispatch: %s, 40-atom chain truncated to "
          "N_prod=2000, 1024 frequencies" % PROFILE_STEP, "",
          "Commands (repository root, one MI355X; OUT is any output directory):", "", "```",
          "rocprofv3 --pmc MfmaUtil MfmaFlopsF64 -d $OUT/pmc_mfma -o run --output-format csv -- python3 "
          "bench.py --forms %s --steps 1 --warmup 0 --no-cpu-baseline --no-serving" % PROFILE_FORM,
          "python bench.py --summarize-mfma $OUT/pmc_mfma/run_counter_collection.csv", "```", "",
          "MfmaUtil = MFMA busy cycles / (active cycles x SIMDs) in percent; MfmaFlopsF64 = executed FP64 matrix "
          "flops (512 per counted op), padding of partial tiles included.", "",
          "| kernel | dispatches | MfmaUtil % | MfmaFlopsF64 per dispatch |", "|---|---:|---:|---:|"]
    for k, cnt, util, fl in rows:
        short = k.replace("(anonymous namespace)::", "")
        short = short.split("(")[0] if "(" in short else short
        short = short[5:] if short.startswith("void ") else short
        md.append("| `%s` | %d | %.1f | %.3e |" % (short[:70], cnt, util, fl))
    with open(out_md, "w") as f:
        f.write("\n".join(md) + "\n")
    print("wrote", out_md)


TRACE_FORMS = {
    # form: (step, calls, note, output file)
    "fp64_A": (PROFILE_STEP, "gw_build_A + gw_solve_W_A",
               "The histogram's bin ranges run on the context's second stream beside the v a0 products, and the "
               "lone point j = 0 is factorised there beside the first frequency batch, so those kernels' durations "
               "include time they share the CUs with each other.", "kernels_fp64A_chain40_n2000.md"),
    "fp64": ("FP64 step (chi0 build + W solve)", "gw_build_chi0 + gw_solve_W",
             "The lone point j = 0 is factorised on the context's second stream beside the first frequency batch, "
             "so the durations of kernels running then include time they share the CUs.",
             "kernels_fp64_chain40_n2000.md"),
}


def summarize_trace(stats_csv, form=PROFILE_FORM):
    """Kernel table from a rocprofv3 --kernel-trace --stats run of the
    profiled step (one warm-up step and one timed step) of one form."""
    step, calls_text, note, fname = TRACE_FORMS[form]
    out_md = os.path.join(HERE, "profiles", fname)
    rows = []
    for r in _csv_rows(stats_csv):
        name = r.get("Name") or r.get("KernelName") or ""
        calls = int(float(r.get("Calls", 0)))
        tot = float(r.get("TotalDurationNs", 0.0))
        rows.append((name, calls, tot))
    rows.sort(key=lambda x: -x[2])
    total = sum(x[2] for x in rows) or 1.0
    md = ["# Kernel profile: %s, 40-atom chain truncated to N_prod=2000, "
          "1024 frequencies" % step, "",
          "Command (repository root, one MI355X; OUT is any output directory):", "", "```",
          "rocprofv3 --kernel-trace --stats -d $OUT/prof_n2000 -o run --output-format csv -- python3 bench.py "
          "--forms %s --steps 1 --warmup 1 --no-cpu-baseline --no-serving" % form,
          "python bench.py --summarize-trace $OUT/prof_n2000/run_kernel_stats.csv %s" % form, "```", "",
          "Two steps (one warm-up, one timed) of %s; all kernels from `run_kernel_stats.csv`.  %s" % (calls_text, note),
          "", "| kernel | calls | total ms | avg us | share |", "|---|---:|---:|---:|---:|"]
    for name, calls, tot in rows:
        short = name.replace("(anonymous namespace)::", "")
        short = short.split("(")[0] if "(" in short else short
        short = short[5:] if short.startswith("void ") else short
        md.append("| `%s` | %d | %.1f | %.1f | %.1f%% |" % (short[:70], calls, tot / 1e6, tot / 1e3 / max(calls, 1),
                                                        100.0 * tot / total))
    md.append("| **all kernels** | | %.1f | | 100%% |" % (total / 1e6))
    with open(out_md, "w") as f:
        f.write("\n".join(md) + "\n")
    print("wrote", out_md)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="n2000", choices=["n2000", "n2000_2w", "n2000_time", "n2000_sigma", "c1", "c2",
                                                                  "c2pair", "c3", "c4"])
    ap.add_argument("--forms", default=None, help="comma list of fp64, fp32_ir, bf16x_ir; n2000 and c1 also "
                    "take the same with _A (A = 1 - v chi0 formed from v a0, then W from A)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--mols", type=int, default=64, help="c3: number of molecules")
    ap.add_argument("--rate", type=float, default=20.0, help="c4: offered requests/s")
    ap.add_argument("--low-rate", type=float, default=0.3, help="c4: the below-capacity run")
    ap.add_argument("--duration", type=float, default=60.0, help="c4: arrival window (s)")
    ap.add_argument("--pool", type=int, default=32, help="c4: molecules at log-spaced atom counts (each arrival "
                    "is served the one nearest its own drawn count)")
    ap.add_argument("--no-serving", action="store_true", help="n2000: skip the bounded serving legs")
    ap.add_argument("--serve-duration", type=float, default=20.0, help="n2000: arrival window of each serving leg (s)")
    ap.add_argument("--serve-pool", type=int, default=16, help="n2000: molecules in the serving pool")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="end with three plain 1 GiB device copies (reference for the HBM counters)")
    ap.add_argument("--summarize-counters", nargs=3, metavar=("STATS_CSV", "FETCH_CSV", "WRITE_CSV"),
                    help="write profiles/hbm_traffic.json from rocprofv3 outputs and exit (no GPU)")
    ap.add_argument("--summarize-mfma", metavar="COUNTER_CSV",
                    help="write profiles/mfma_chain40_n2000.md from a MfmaUtil/MfmaFlopsF64 counter run")
    ap.add_argument("--summarize-trace", nargs="+", metavar="STATS_CSV [FORM]",
                    help="write the kernel table of one form (fp64_A, the default, or fp64) to "
                         "profiles/kernels_<form>_chain40_n2000.md and exit (no GPU)")
    args = ap.parse_args()
    if args.summarize_mfma:
        summarize_mfma(args.summarize_mfma, os.path.join(HERE, "profiles", "mfma_chain40_n2000.md"))
        return
    if args.summarize_trace:
        summarize_trace(*args.summarize_trace[:2])
        return
    if args.summarize_counters:
        summarize_profiles(*args.summarize_counters, TRAFFIC_FILE)
        return
    if args.gpus != 1:
        print("bench.py measures one GPU: the library has no multi-GPU path (the sharding design is "
              "documented, not built); run with --gpus 1", file=sys.stderr)
        sys.exit(2)
    if args.forms is None:
        args.forms = {"n2000": "fp64,fp64_A,fp32_ir,bf16x_ir,fp32_ir_A,bf16x_ir_A", "n2000_2w": "fp64",
                      "n2000_time": "fp64",
                      "n2000_sigma": "fp64",
                      "c1": "fp64,fp64_A,bf16x_ir",
                      "c2": "fp64,fp64_A,bf16x_ir,bf16x_ir_A",
                      "c2pair": "fp64", "c3": "fp64", "c4": "fp64"}[args.workload]

    import torch

    sys.path.insert(0, HERE)
    import gw_synth as gs
    import paper_1101_2065_amd.gw as gw

    if args.workload == "n2000":
        log("generating molecule")
        mol = gs.truncate_products(gs.make_config(1), N_PROD)
        out = run_single(args, gw, gs, torch, mol, gs.config_grid(1), "chain40_nprod2000_nomega1024")
    elif args.workload == "n2000_2w":
        out = run_two_window(args, gw, gs, torch)
    elif args.workload == "n2000_time":
        out = run_time_route(args, gw, gs, torch)
    elif args.workload == "n2000_sigma":
        out = run_self_energy(args, gw, gs, torch)
    elif args.workload == "c1":
        log("generating molecule")
        mol = gs.make_config(1)
        out = run_single(args, gw, gs, torch, mol, gs.config_grid(1), "chain40_nprod%d_nomega1024" % mol.n_prod)
    elif args.workload == "c2":
        out = run_c2(args, gw, gs, torch)
    elif args.workload == "c2pair":
        out = run_c2pair(args, gw, gs, torch)
    elif args.workload == "c3":
        out = run_c3(args, gw, gs, torch)
    else:
        out = run_c4(args, gw, gs, torch)
    if args.copy_calibration:
        a = torch.empty(COPY_BYTES // 8, dtype=torch.float64, device="cuda").fill_(1.0)
        b = torch.empty_like(a)
        for _ in range(3):
            torch.mul(a, 1.0, out=b)  # one kernel: reads and writes COPY_BYTES
        torch.cuda.synchronize()
        log("copy calibration: 3 x %d bytes" % COPY_BYTES)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
