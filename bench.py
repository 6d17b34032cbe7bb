#!/usr/bin/env python3
"""Benchmark of the deflated-CG solve on one MI355X.

Workload (the headline configuration): unit square, 512 x 512 squares,
DG-Q1 pseudo-stress (4,194,304 unknowns), dt = 1e-4, nu = 1, penalty 10/h,
RHS b ~ N(0, 1) from a seed, tol 1e-8 on the true residual (at most two warm
restarts of Algorithm 2 when the recurrence test stops above it), c_F =
0.01, W-cycle with 2 + 2 RAS sweeps on four levels, mixed form (FP32
multigrid inside the FP64 deflated CG).  A step is one complete dcg_solve
(prologue, all outer iterations, epilogue) with all operators and vectors
resident in HBM; ``value`` is solves per second.

Also reported on the same JSON line:
  roofline      the dominant kernel (finest-level RAS step, grouped MFMA
                kernel): algorithmic flops per launch / average launch time
                measured with HIP events inside the timed solves, against the
                FP32 matrix peak; its HBM bytes and rate beside
  err_vs_oracle the same configuration against the CPU oracle's golden files
  fp64          the all-FP64 form on seed 0, against the mixed seed-0 solve
  inner_tolerance_variants_seed0  c_F = 1e-4 and the adaptive rule (eq. (tol))
  cpu_baseline  the CPU oracle on a bounded sample of the same workload
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
def astar_bytes(n):
    """Algorithmic HBM bytes of one k_astar launch with the fused direction
    update (2D): r and p read, p and w written (4 x 128 B) and s = Z^T w (32 B)
    per square; the operator is a table of its class blocks, read from cache."""
    return (4 * 128 + 32) * n * n


def copy_gbs(nbytes=1 << 30, reps=10):
    """Bandwidth of a plain device-to-device copy (read + write bytes / time),
    the practical ceiling next to the vendor peak."""
    import torch
    a = torch.empty(nbytes // 8, dtype=torch.float64, device="cuda")
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
    gbs = 2 * nbytes * reps / (e0.elapsed_time(e1) * 1e-3) / 1e9
    del a, b
    torch.cuda.empty_cache()
    return gbs


def sweep_bytes_per_square(s):
    """Algorithmic HBM bytes per square of one RAS step, element size s, as
    the mean over the four steps of a level visit (zero start, two with the
    pending update, one with the prolongation).  Every step reads f and
    writes the tile outputs (128 per 16-square core); all but the first read
    the square's iterate and write the resolved iterate; the pending outputs
    (12 per square) or the coarse iterate and its pending outputs (a quarter
    square's worth) come on top.  The tile inverses and the level operator
    are not charged per square: on the uniform grid they fall into 9 classes
    each (3 x 3 tile and square positions), read once per launch
    (sweep_launch_bytes); the pending slots and weights follow from the
    geometry and cost no bytes."""
    base = 4 * s + 8 * s
    zero = base
    pending = base + 4 * s + 12 * s + 4 * s
    prolong = base + 4 * s + 4 * s + (4 * s + 12 * s) / 4
    return (zero + 2 * pending + prolong) / 4


# The finest-level RAS launches of every TIMING_STRIDE-th W-cycle are bracketed
# by HIP events during the timed solve: an event pair costs a few microseconds of
# stream time, which timing all launches of a solve would add to it.
TIMING_STRIDE = 8

SWEEP_CLASSES = 9    # distinct RAS local problems and operator rows per level
FP32_MFMA_PEAK_TFS = 157.3   # MI355X dense FP32 matrix peak
FP64_VECTOR_PEAK_TFS = 78.6   # MI355X FP64 vector peak (FMA)


def sweep_launch_bytes(n, s):
    """Algorithmic bytes of one RAS step on a level of n x n squares: the
    per-square vectors and, once, the 9 class inverses (full 128 x 128, in
    MFMA operand order) and the 9 class rows of the level operator."""
    return int(sweep_bytes_per_square(s) * n * n + SWEEP_CLASSES * (128 * 128 + 80) * s)


def sweep_launch_flops(n):
    """Algorithmic flops of one RAS step on a level of n x n squares: the
    tile solves (a 128 x 128 inverse times a 128-vector per tile) and the
    residual (80 multiply-adds per square)."""
    tiles = (n // 4) ** 2
    return tiles * 2 * 128 * 128 + n * n * 2 * 80


def sweep_l2_factor_bytes(n, s, group=4):
    """Bytes of class inverse one grouped RAS launch reads from L2: every
    workgroup (a group of group x group tiles, one per class present) reads
    the whole 128 x 128 inverse of its class."""
    gpr = n // 4 // group
    boundary_extra = 4 * (gpr - 2) + 3 * 4 if gpr >= 2 else 8   # edge groups 2 classes, corners 4
    return (gpr * gpr + boundary_extra) * 128 * 128 * s


def read_golden(name):
    """Counts and the sampled x of an oracle golden file (tests/golden)."""
    import numpy as np
    meta, idx, val = {}, [], []
    with open(os.path.join(ROOT, "tests", "golden", name)) as fh:
        for line in fh:
            if line.startswith("#") or not line.strip():
                continue
            k, v = line.split()
            if k.isdigit():
                idx.append(int(k))
                val.append(float(v))
            else:
                meta[k] = float(v)
    return meta, np.array(idx), np.array(val)


def err_vs_oracle(dcg):
    """The benchmark's configuration (four levels, dt = 1e-4, tol 1e-8,
    c_F = 0.01, seed 0) against the CPU FP64 oracle's golden files: the
    iterate after the first 30 outer iterations at n = 512 (the whole oracle
    solve at this size takes days on the CPU) and the whole solve at n = 256;
    relative ell2 error over the 4096 entries each file holds, both forms."""
    import numpy as np
    import torch
    from dcg_workloads import rhs
    out = {}
    for key, name, n, max_outer, restarts in (
            ("n512_first_30_outer", "headline_n512_J4_seed0_out30.txt", 512, 30, 0),
            ("n256_whole_solve", "headline_n256_J4_seed0.txt", 256, 100000, 2)):
        meta, idx, val = read_golden(name)
        res = {"oracle_outer": int(meta["outer"]), "oracle_total_wcycles": int(meta["total_cycles"])}
        for prec in ("mixed", "fp64"):
            s = dcg.Solver(n, 1e-4, prec=prec, levels=4, max_outer=max_outer, restarts=restarts)
            b = torch.from_numpy(rhs(n, 0)).cuda()
            x = torch.empty_like(b)
            _, st = s.solve(b, x, 1e-8)
            xs = x.cpu().numpy()[idx]
            res[prec] = {"rel_err": float(np.linalg.norm(xs - val) / np.linalg.norm(val)),
                         "outer": st.outer_iters, "total_wcycles": st.total_wcycles}
            s.close()
        out[key] = res
        log("err vs oracle %s: mixed %.2e, fp64 %.2e" % (key, res["mixed"]["rel_err"], res["fp64"]["rel_err"]))
    return out


# HBM traffic of one finest-level RAS launch at n = 512 (mixed form), from two
# rocprofv3 --pmc runs (FETCH_SIZE, WRITE_SIZE; profiles/k_sweep_g_finest_n512_mixed_traffic.md),
# each scaled by the reading of a plain 1 GiB copy (FETCH_SIZE reads 0.5 GiB for it, WRITE_SIZE
# 1 GiB).  Valid only for the kernel source it was taken on: the digest of the RAS kernel
# sources must match, else the bench reports traffic as null.
TRAFFIC = {"source_digest": "6aa698dd3cb9d588", "n": 512,
           "fetch_kib": 9365.8, "fetch_scale": 2.0, "write_kib": 14646.3, "write_scale": 1.0}


def kernel_source_digest():
    import hashlib
    h = hashlib.sha256()
    for f in ("mg_kernels.hip", "mg_common.hpp"):
        with open(os.path.join(ROOT, "paper_2606_13429_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(n):
    """HBM bytes per finest RAS launch from the counters, or None when they
    do not apply (other n, or the kernel changed since they were taken)."""
    try:
        if n != TRAFFIC["n"] or kernel_source_digest() != TRAFFIC["source_digest"]:
            return None
    except OSError:
        return None
    return int(1024 * (TRAFFIC["fetch_kib"] * TRAFFIC["fetch_scale"]
                       + TRAFFIC["write_kib"] * TRAFFIC["write_scale"]))


def levels_option(n, levels):
    """dcg_options.levels for a requested depth: 0 (the whole stored hierarchy)
    when the mesh has no more than ``levels`` levels."""
    from paper_2606_13429_amd import _binding as lib
    return 0 if levels <= 0 or levels >= lib.dcg_num_levels(n) else levels


def log(msg):
    print("[bench] " + msg, file=sys.stderr, flush=True)


def cpu_baseline(n, dt, tol, gpu_outer, gpu_wcycles, c_F=0.01):
    """The CPU oracle (FP64, NumPy/SciPy) on a bounded sample of the same
    solve: one inner Multigrid solve (the prologue's, Algorithm 3 to c_F tol)
    and one A* product, timed; solves/s extrapolated with the GPU solve's
    W-cycle and outer-iteration counts (each outer iteration applies A*
    twice in the oracle's M_D).  Oracle setup is not counted."""
    from dcg_workloads import rhs
    from oracle import discretisation, multigrid
    t0 = time.time()
    As = discretisation.operator(n, dt)
    V = discretisation.deflation_basis(n)
    E = (V.T @ As @ V).tocsr()
    H = multigrid.Hierarchy(E, n)
    t_setup = time.time() - t0
    b = rhs(n, 0).reshape(n * n, 4, 4).transpose(1, 0, 2).reshape(-1)
    s = V.T @ b
    t0 = time.time()
    _, cycles = multigrid.multigrid(H, s, tol=c_F * tol)
    t_inner = time.time() - t0
    t0 = time.time()
    w = As @ b
    t_spmv = time.time() - t0
    t_wcycle = t_inner / max(cycles, 1)
    t_solve = gpu_wcycles * t_wcycle + 2 * (gpu_outer + 2) * t_spmv
    threads = os.environ.get("OMP_NUM_THREADS") or str(os.cpu_count())
    return {"value": 1.0 / t_solve, "unit": "solves/s", "cores": int(threads),
            "kind": "oracle",
            "sample": ("n=%d dt=%g: one inner multigrid solve on the oracle's full hierarchy "
                       "(coarsest 16x16, dense Cholesky; %d W-cycles, %.1f s) and one A* product "
                       "(%.2f s), extrapolated to the GPU solve's %d W-cycles and %d outer iterations "
                       "(estimate %.0f s per solve); oracle setup %.0f s not counted"
                       % (n, dt, cycles, t_inner, t_spmv, gpu_wcycles, gpu_outer, t_solve, t_setup)),
            "seconds_per_solve": t_solve}


def serving_cpu_estimate(per_request, tol, c_F=0.01):
    """The CPU oracle's cost of the trace, estimated: per mesh size, one inner
    multigrid solve and one A* product are timed; each request is charged its
    GPU-measured W-cycles and outer iterations at those rates."""
    from dcg_workloads import rhs
    from oracle import discretisation, multigrid
    rates = {}
    for n in sorted({r["n"] for r in per_request}):
        As = discretisation.operator(n, 1e-4)
        V = discretisation.deflation_basis(n)
        H = multigrid.Hierarchy((V.T @ As @ V).tocsr(), n)
        b = rhs(n, 0).reshape(n * n, 4, 4).transpose(1, 0, 2).reshape(-1)
        t0 = time.time()
        _, cycles = multigrid.multigrid(H, V.T @ b, tol=c_F * tol)
        t_w = (time.time() - t0) / max(cycles, 1)
        t0 = time.time()
        As @ b
        rates[n] = (t_w, time.time() - t0)
        log("oracle rates n=%d: %.3f s per W-cycle, %.3f s per A* product" % (n, *rates[n]))
    total = sum(r["wcycles"] * rates[r["n"]][0] + 2 * (r["outer"] + 2) * rates[r["n"]][1]
                for r in per_request)
    threads = os.environ.get("OMP_NUM_THREADS") or str(os.cpu_count())
    return {"value": len(per_request) / total, "unit": "solves/s", "cores": int(threads),
            "kind": "oracle",
            "sample": "per mesh size one oracle inner multigrid solve and one A* product timed; "
                      "every request charged its GPU-measured W-cycles and outer iterations "
                      "(estimate %.0f s for the trace, requests run back to back)" % total}


def converged_stats(done, makespan, ok):
    """Throughput and latency over the requests that met tol: solves that
    converged per second of the trace's makespan, p50 / p99 of their latency."""
    import numpy as np
    conv = [d for d in done if d["status"] == ok]
    if not conv:
        return None
    lat = np.array([d["latency"] for d in conv])
    return {"requests": len(conv), "solves_per_s": round(len(conv) / makespan, 3),
            "p50_latency_s": round(float(np.percentile(lat, 50)), 3),
            "p99_latency_s": round(float(np.percentile(lat, 99)), 3),
            "max_rel_res_true": max(d["rel_res_true"] for d in conv)}


def serving(args):
    """The serving workload: a Poisson trace of requests replayed in real time
    against one dcg server; latency = arrival to completion."""
    import numpy as np
    import torch
    import paper_2606_13429_amd as dcg
    from paper_2606_13429_amd import _binding as lib
    from dcg_workloads import SERVING, rhs, serving_trace

    sizes = tuple(SERVING["sizes"])
    trace = serving_trace(seed=0, count=args.requests, rate=SERVING["rate"], sizes=sizes,
                          dt_range=SERVING["dt_range"])
    tol = SERVING["tol"]
    torch.cuda.set_device(0)
    srv = dcg.Server(prec="mixed", max_outer=args.serve_max_outer, c_A=args.serve_c_A)
    t0 = time.time()
    for n in sizes:
        srv.prepare(n)
    log("contexts for n=%s prepared in %.1f s" % (list(sizes), time.time() - t0))
    bs = [torch.from_numpy(rhs(r["n"], r["seed"])).cuda() for r in trace]
    xs = [torch.empty_like(b) for b in bs]
    torch.cuda.synchronize()
    pending, done = {}, [None] * len(trace)
    t_start = time.perf_counter()
    last_log = t_start
    i = 0
    while i < len(trace) or pending:
        now = time.perf_counter() - t_start
        while i < len(trace) and trace[i]["t_arrival"] <= now:
            r = trace[i]
            pending[srv.submit(r["n"], r["dt"], bs[i], xs[i], tol)] = i
            i += 1
        for tk in list(pending):
            status, st = srv.poll(tk)
            if status == lib.DCG_PENDING:
                continue
            k = pending.pop(tk)
            if status < 0:
                log("request %d (n=%d dt=%.3g) failed: status %d, %s"
                    % (k, trace[k]["n"], trace[k]["dt"], status, lib.dcg_last_error()))
            done[k] = dict(n=trace[k]["n"], dt=trace[k]["dt"], status=status,
                           outer=st.outer_iters, wcycles=st.total_wcycles,
                           latency=time.perf_counter() - t_start - trace[k]["t_arrival"],
                           queue_ms=st.t_queue_ms, rel_res_true=st.rel_res_true)
        if time.perf_counter() - last_log > 10.0:
            last_log = time.perf_counter()
            log("t=%.0f s: %d submitted, %d done" % (last_log - t_start, i, sum(d is not None for d in done)))
        time.sleep(2e-4)
    makespan = time.perf_counter() - t_start
    steps, slot_steps = srv.counters()
    lat = np.array([d["latency"] for d in done])
    capped = [d for d in done if d["status"] == lib.DCG_NOT_CONVERGED]
    failed = [d for d in done if d["status"] < 0]
    per_n = {}
    for n in sizes:
        ds = [d for d in done if d["n"] == n]
        if not ds:
            continue
        ln = np.array([d["latency"] for d in ds])
        per_n[str(n)] = {"requests": len(ds),
                         "not_converged": sum(d["status"] == lib.DCG_NOT_CONVERGED for d in ds),
                         "p50_latency_s": round(float(np.percentile(ln, 50)), 3),
                         "p99_latency_s": round(float(np.percentile(ln, 99)), 3),
                         "mean_outer": round(float(np.mean([d["outer"] for d in ds])), 1),
                         "mean_wcycles": round(float(np.mean([d["wcycles"] for d in ds])), 1)}
    # a request alone in a fresh server gives bitwise the same x and counts
    probe = int(np.argmin([d["wcycles"] if d["status"] == lib.DCG_OK and d["n"] == 64 else 1 << 30
                           for d in done]))
    alone = dcg.Server(prec="mixed", max_outer=args.serve_max_outer, c_A=args.serve_c_A)
    xa = torch.empty_like(xs[probe])
    r = trace[probe]
    status, st = alone.wait(alone.submit(r["n"], r["dt"], bs[probe], xa, tol))
    alone_ok = bool(torch.equal(xa, xs[probe])) and st.outer_iters == done[probe]["outer"]
    alone.close()
    result = {
        "metric": "dCG serving: solves/s and p50/p99 latency (arrival to done) over a Poisson trace",
        "value": round(len(done) / makespan, 3), "unit": "solves/s", "n_gpus": 1,
        "steps": len(trace), "warmup": 0, "ms_per_step": round(1000 * makespan / len(trace), 2),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f64 outer / f32 multigrid", "data": "synthetic: serving trace seed 0",
        "config": {"workload": "serving trace: %d requests, Poisson %.0f/s, n in %s, dt 10^U%s, "
                               "tol %g, mixed form, max_outer %d, inner tolerance %s"
                               % (len(trace), SERVING["rate"], list(sizes), tuple(SERVING["dt_range"]),
                                  tol, args.serve_max_outer,
                                  "adaptive c_A=%g" % args.serve_c_A if args.serve_c_A else "fixed c_F=0.01")},
        "p50_latency_s": round(float(np.percentile(lat, 50)), 3),
        "p99_latency_s": round(float(np.percentile(lat, 99)), 3),
        "converged_only": converged_stats(done, makespan, lib.DCG_OK),
        "capped": [{"n": d["n"], "dt": round(d["dt"], 8), "outer": d["outer"],
                    "rel_res_true": d["rel_res_true"], "latency_s": round(d["latency"], 2)}
                   for d in capped],
        "makespan_s": round(makespan, 2), "not_converged": len(capped), "failed": len(failed),
        "failures": [{"n": d["n"], "dt": d["dt"], "status": d["status"]} for d in failed],
        "batch_occupancy": round(slot_steps / max(steps, 1), 2), "server_steps": steps,
        "per_n": per_n, "alone_vs_mix_bitwise": alone_ok,
    }
    srv.close()
    if not args.skip_cpu:
        result["cpu_baseline"] = serving_cpu_estimate(done, tol)
    print(json.dumps(result), flush=True)


def dt_sweep(args):
    """Outer iterations, Tot and Inn against dt at n = 128 (the FP64 form with
    the full preconditioner; the mixed form beside it), one solve each, and
    the finest-level RAS step's event-timed rate."""
    import torch
    import paper_2606_13429_amd as dcg
    from paper_2606_13429_amd import _binding as lib
    from dcg_workloads import rhs
    n, tol = args.sweep_n, args.tol
    torch.cuda.set_device(0)
    b = torch.from_numpy(rhs(n, 0)).cuda()
    x = torch.empty_like(b)
    rows = []
    s_bytes = {"fp64": 8, "mixed": 4}
    dts = [float(v) for v in args.sweep_dts.split(",")]
    for dt in dts:
        for prec in args.sweep_precs.split(","):
            solver = dcg.Solver(n, dt, prec=prec, max_outer=args.sweep_max_outer, c_F=args.sweep_cF)
            solver.solve(b, x, tol)                      # warm-up (graph capture)
            lib.dcg_kernel_timing(solver.handle, True)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            status, st = solver.solve(b, x, tol)
            torch.cuda.synchronize()
            t = time.perf_counter() - t0
            k_ms, k_n = lib.dcg_kernel_timing_read(solver.handle)
            solver.close()
            gbs = sweep_launch_bytes(n, s_bytes[prec]) / (k_ms / max(k_n, 1) * 1e-3) / 1e9
            rows.append({"dt": dt, "form": prec, "status": status, "outer": st.outer_iters,
                         "tot": st.total_wcycles, "inn": round(st.inner_per_outer, 2),
                         "solve_s": round(t, 3), "rel_res_true": st.rel_res_true,
                         "finest_ras_us": round(k_ms / max(k_n, 1) * 1e3, 2),
                         "finest_ras_GBs": round(gbs, 1)})
            log("dt=%g %s: status %d outer %d Tot %d Inn %.2f %.2f s, finest RAS %.1f us"
                % (dt, prec, status, st.outer_iters, st.total_wcycles, st.inner_per_outer, t,
                   rows[-1]["finest_ras_us"]))
        # the comparison of Tables 1-2: plain CG (no deflation) and deflated CG with an
        # exact inner solve on the same system
        for inner in ("none", "exact"):
            solver = dcg.Solver(n, dt, prec="fp64", inner=inner, max_outer=args.sweep_max_outer)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            status, st = solver.solve(b, x, tol)
            torch.cuda.synchronize()
            t = time.perf_counter() - t0
            solver.close()
            rows.append({"dt": dt, "form": "fp64", "inner": inner, "status": status,
                         "outer": st.outer_iters, "solve_s": round(t, 3), "rel_res_true": st.rel_res_true})
            log("dt=%g %s: status %d outer %d %.2f s" % (dt, "plain CG" if inner == "none" else "DCG exact inner",
                                                          status, st.outer_iters, t))
    print(json.dumps({"metric": "dCG outer iterations / Tot / Inn against dt", "n": n, "tol": tol,
                      "c_F": args.sweep_cF, "max_outer": args.sweep_max_outer, "rows": rows}),
          flush=True)


def timestep(args):
    """BDF2 time stepping at n = 1024 (mixed form, warm start): steps/s and
    the true residual of every step, over --ts-steps steps."""
    import numpy as np
    import torch
    from paper_2606_13429_amd import _binding as lib
    from paper_2606_13429_amd.timestep import BDF2
    from dcg_workloads import TIMESTEP, forcing_load, fourier_modes
    n, dt = TIMESTEP["n"], TIMESTEP["dt"]
    torch.cuda.set_device(0)
    t0 = time.time()
    F = torch.from_numpy(forcing_load(n, fourier_modes(TIMESTEP["seed"], TIMESTEP["modes"]))).cuda()
    kw = {}
    if args.ts_outer_mg > 0:   # the outer multigrid preconditioner (another method, reading 25)
        kw = dict(outer="fcg", m_max=8, outer_mg=args.ts_outer_mg)
    stepper = BDF2(n, dt, prec="mixed", tol=args.tol, levels=levels_option(n, args.levels), **kw)
    log("n=%d setup + forcing %.1f s" % (n, time.time() - t0))
    lib.dcg_kernel_timing(stepper.solver.handle, TIMING_STRIDE)
    rows = []
    torch.cuda.synchronize()
    t_all = time.perf_counter()
    for i in range(args.ts_steps):
        t0 = time.perf_counter()
        st = stepper.step(F)
        torch.cuda.synchronize()
        rows.append({"step": i + 1, "status": st.status, "outer": st.outer_iters,
                     "tot": st.total_wcycles, "rel_res_true": st.rel_res_true,
                     "seconds": round(time.perf_counter() - t0, 3)})
        log("step %d: outer %d Tot %d res %.2e %.1f s" % (i + 1, st.outer_iters, st.total_wcycles,
                                                           st.rel_res_true, rows[-1]["seconds"]))
    t_all = time.perf_counter() - t_all
    k_ms, k_n = lib.dcg_kernel_timing_read(stepper.solver.handle)
    k_avg = k_ms / max(k_n, 1)
    tflops = sweep_launch_flops(n) / (k_avg * 1e-3) / 1e12
    gbs = sweep_launch_bytes(n, 4) / (k_avg * 1e-3) / 1e9
    method = ("deflated CG" if args.ts_outer_mg <= 0 else
              "FCG(8) with the outer multigrid preconditioner, m = %d" % args.ts_outer_mg)
    print(json.dumps({"metric": "BDF2 steps/s, n=1024 dt=1e-5, mixed form, warm start",
                      "method": method,
                      "value": round(len(rows) / t_all, 5), "unit": "steps/s", "steps": len(rows),
                      "of_steps": TIMESTEP["steps"], "seconds": round(t_all, 2),
                      "roofline": {"bound": "mfma", "kernel": "k_sweep_g<float,4> (finest-level RAS step)",
                                   "achieved": round(tflops, 2), "peak": FP32_MFMA_PEAK_TFS,
                                   "unit": "TFLOP/s", "frac": round(tflops / FP32_MFMA_PEAK_TFS, 4),
                                   "flops_per_launch": sweep_launch_flops(n),
                                   "hbm_achieved_gbs": round(gbs, 1),
                                   "hbm_frac": round(gbs / HBM_PEAK_GBS, 4),
                                   "avg_launch_us": round(k_avg * 1e3, 2), "launches": k_n},
                      "rows": rows}), flush=True)


def lap3_bytes(n):
    """Algorithmic HBM bytes of one k_lap3 launch (the inner Laplacian of the
    3D solver): the 8 x 8 FP64 blocks that exist (the element and its face
    neighbours inside the cube) plus p read and q written once."""
    ne = n ** 3
    nblocks = ne + 6 * n * n * (n - 1)
    return 8 * (64 * nblocks + 16 * ne)


def astar3_bytes(n):
    """Algorithmic HBM bytes of one k_astar3 launch (the 3D A* product): x read
    and y written once (72 FP64 values per cube each); the operator is a table of
    its class blocks, read from cache."""
    return 8 * 144 * n ** 3


def mg3_ras_flops(n):
    """Algorithmic flops of one finest-level RAS step of the 3D multigrid
    (k_mg3_ras): per cube 8 rows times 8 values of every diamond cube inside
    the domain (the cube's blocks' solutions restricted to it, combined into
    one 8 x 200 update per class), two flops per multiply-add."""
    import numpy as np
    x = np.arange(n)
    total = 0
    for dz in range(-2, 3):
        for dy in range(-2, 3):
            for dx in range(-2, 3):
                if abs(dx) + abs(dy) + abs(dz) > 2:
                    continue
                cnt = [int(((x + d >= 0) & (x + d < n)).sum()) for d in (dx, dy, dz)]
                total += cnt[0] * cnt[1] * cnt[2]
    return 2 * 64 * total


def mg3_ras_bytes(n):
    """Algorithmic bytes of one finest-level RAS step of the 3D multigrid:
    r read and z read and written once (8 FP64 values per cube each), plus
    the class tables the level holds (343 x 8 x 200 FP64), read once."""
    return 8 * (24 * n ** 3 + 343 * 8 * 200)


def three_d(args):
    """The 3D solver (d = 3 block structure) at n^3 = 32^3 cubes, dt = 1e-3,
    FP64, with the exact inner solve (fast diagonalisation, the setting of
    Table 5 left), the multigrid inner solve (--3d-inner mg: W-cycles with the
    RAS smoother, m = 10, Table 5 right; --3d-cA for the adaptive rule) or
    block-Jacobi CG (--3d-inner cg): solves/s, outer and inner counts, and the
    roofline of the dominant kernel (A*, the finest RAS step, resp. the inner
    Laplacian product), timed with HIP events inside the library."""
    import torch
    import paper_2606_13429_amd as dcg
    from paper_2606_13429_amd import _binding as lib
    from dcg_workloads import THREE_D, rhs3d
    n, dt, tol = args.n3, THREE_D["dt"], THREE_D["tol"]
    torch.cuda.set_device(0)
    t0 = time.time()
    s = dcg.Solver3D(n, dt, nu=THREE_D["nu"], penalty=THREE_D["penalty"], inner=args.inner3,
                     c_A=args.cA3, max_outer=args.max_outer3, levels=args.levels3,
                     restarts=args.restarts3)
    log("3d setup n=%d (%d elements) %.1f s" % (n, n ** 3, time.time() - t0))
    bs = [torch.from_numpy(rhs3d(n, i)).cuda() for i in range(max(args.steps, 1))]
    x = torch.empty_like(bs[0])
    for i in range(args.warmup):
        st = s.solve(bs[0], x, tol)[1]
        log("3d warmup %d: outer=%d inner steps=%d %.1f ms" % (i, st.outer_iters, st.total_wcycles,
                                                                 st.t_solve_ms))
    lib.dcg3d_kernel_timing(s.handle, True)
    rows = []
    torch.cuda.synchronize()
    t_all = time.perf_counter()
    for i in range(args.steps):
        status, st = s.solve(bs[i], x, tol)
        rows.append({"status": status, "outer": st.outer_iters, "restarts": st.restarts,
                     "inner_steps": st.total_wcycles,
                     "inner_per_outer": round(st.inner_per_outer, 2), "rel_res_true": st.rel_res_true,
                     "ms": round(st.t_solve_ms, 1)})
        log("3d step %d: status=%d outer=%d inner steps=%d res=%.2e %.1f ms"
            % (i, status, st.outer_iters, st.total_wcycles, st.rel_res_true, st.t_solve_ms))
    torch.cuda.synchronize()
    t_all = time.perf_counter() - t_all
    k_ms, k_n = lib.dcg3d_kernel_timing_read(s.handle)
    lib.dcg3d_kernel_timing(s.handle, False)
    k_avg = k_ms / max(k_n, 1)
    inner_name = {"exact": "exact (fast diagonalisation)", "cg": "block-Jacobi CG",
                  "mg": "W-cycle multigrid, RAS, m = 10, %s" % (
                      "adaptive c_A=%g" % args.cA3 if args.cA3 else "fixed c_F=0.01")}[args.inner3]
    if args.inner3 == "mg":
        flops = mg3_ras_flops(n)
        nbytes = mg3_ras_bytes(n)
        tfs = flops / (k_avg * 1e-3) / 1e12
        gbs = nbytes / (k_avg * 1e-3) / 1e9
        roof = {"bound": "mfma", "kernel": "k_mg3_ras (finest-level RAS step, FP64 MFMA)",
                "achieved": round(tfs, 3), "peak": FP64_VECTOR_PEAK_TFS, "unit": "TFLOP/s",
                "frac": round(tfs / FP64_VECTOR_PEAK_TFS, 4), "traffic": None,
                "flops_per_launch": flops, "bytes_per_launch": nbytes,
                "hbm_achieved_gbs": round(gbs, 1), "hbm_frac": round(gbs / HBM_PEAK_GBS, 4),
                "avg_launch_us": round(k_avg * 1e3, 2), "launches": k_n}
    else:
        exact = args.inner3 == "exact"
        nbytes = astar3_bytes(n) if exact else lap3_bytes(n)
        kname = "k_astar3 (A* product)" if exact else "k_lap3 (inner Laplacian product)"
        gbs = nbytes / (k_avg * 1e-3) / 1e9
        roof = {"bound": "hbm", "kernel": kname,
                "achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(gbs / HBM_PEAK_GBS, 4),
                "traffic": None,
                "avg_launch_us": round(k_avg * 1e3, 2), "launches": k_n,
                "bytes_per_launch": nbytes}
    print(json.dumps({
        "metric": "3D dCG solves/s, %d^3 DG-Q1 cubes, dt=%g, FP64, inner %s" % (n, dt, inner_name),
        "value": round(args.steps / t_all, 5), "unit": "solves/s", "steps": args.steps,
        "warmup": args.warmup, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "3D pseudo-stress A* x = b, n=%d, dt=%g, nu=%g, penalty=%g, tol=%g"
                   % (n, dt, THREE_D["nu"], THREE_D["penalty"], tol)},
        "roofline": roof,
        "mg_levels": list(s.mg_levels()) if args.inner3 == "mg" else None,
        "rows": rows}), flush=True)
    s.close()


def levels_sweep(args):
    """Multigrid depth at the headline size: one warm solve per depth (levels
    2 .. J, coarsest exact by fast diagonalisation, J = dense Cholesky of 16 x
    16 squares), mixed form, capped at --sweep-max-outer outer iterations, so
    that the time per W-cycle and the W-cycle counts can be compared."""
    import torch
    import paper_2606_13429_amd as dcg
    from paper_2606_13429_amd import _binding as lib
    from dcg_workloads import rhs
    n, dt, tol = args.n, args.dt, args.tol
    torch.cuda.set_device(0)
    b = torch.from_numpy(rhs(n, 0)).cuda()
    x = torch.empty_like(b)
    J = lib.dcg_num_levels(n)
    rows = []
    for levels in range(2, J + 1):
        solver = dcg.Solver(n, dt, prec="mixed", max_outer=args.sweep_max_outer,
                            levels=0 if levels == J else levels)
        solver.solve(b, x, tol)                          # warm-up (graph capture)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        status, st = solver.solve(b, x, tol)
        torch.cuda.synchronize()
        t = time.perf_counter() - t0
        solver.close()
        nc = n >> (levels - 1)
        rows.append({"levels": levels, "coarsest": "%dx%d" % (nc, nc), "status": status,
                     "outer": st.outer_iters, "tot": st.total_wcycles,
                     "inn": round(st.inner_per_outer, 2), "solve_ms": round(1e3 * t, 1),
                     "ms_per_wcycle": round(1e3 * t / max(st.total_wcycles, 1), 4)})
        log("levels=%d (coarsest %s): outer %d Tot %d Inn %.2f  %.1f ms, %.3f ms per W-cycle"
            % (levels, rows[-1]["coarsest"], st.outer_iters, st.total_wcycles, st.inner_per_outer,
               1e3 * t, rows[-1]["ms_per_wcycle"]))
    print(json.dumps({"levels_sweep": rows, "n": n, "dt": dt, "tol": tol,
                      "max_outer": args.sweep_max_outer}), flush=True)


def three_d_sweep(args):
    """The 3D analogue of Table 5 (left): deflated-CG outer iterations with the
    exact inner solve against dt on three nested meshes (n = 8, 16, 32 cubes
    per side), tol = 1e-8, one seeded right-hand side per mesh."""
    import torch
    import paper_2606_13429_amd as dcg
    from dcg_workloads import THREE_D, rhs3d
    torch.cuda.set_device(0)
    rows = []
    for n in (8, 16, 32):
        b = torch.from_numpy(rhs3d(n, 0)).cuda()
        x = torch.empty_like(b)
        for dt in (1.0, 0.5, 0.1, 1e-2, 1e-3, 1e-4, 1e-5):
            for inner in ("exact", "none"):      # deflated CG, and plain CG beside it
                s = dcg.Solver3D(n, dt, nu=THREE_D["nu"], penalty=THREE_D["penalty"],
                                 max_outer=args.sweep_max_outer, inner=inner)
                status, st = s.solve(b, x, THREE_D["tol"])
                s.close()
                rows.append({"n": n, "dt": dt, "method": "DCG" if inner == "exact" else "CG",
                             "status": status, "outer": st.outer_iters,
                             "rel_res_true": st.rel_res_true, "ms": round(st.t_solve_ms, 1)})
                log("3d sweep n=%d dt=%g %s: status=%d outer=%d res=%.2e %.1f ms"
                    % (n, dt, rows[-1]["method"], status, st.outer_iters, st.rel_res_true, st.t_solve_ms))
    print(json.dumps({"metric": "3D outer iterations vs dt: DCG (exact inner solve) and plain CG, n = 8, 16, 32",
                      "unit": "iterations", "tol": THREE_D["tol"], "rows": rows}), flush=True)


def outer_mg_sweep(args):
    """The outer multigrid preconditioner against mesh size: per (n, dt) the
    paper's deflated CG (fixed inner tolerance), FCG(8) and FCG(8) with B =
    one W-cycle on A* (m = --omg-m), mixed form, b = rhs(n, 0), tol 1e-8:
    outer iterations, W-cycles, wall time and the true residual."""
    import torch
    import paper_2606_13429_amd as dcg
    from paper_2606_13429_amd import _binding as lib
    from dcg_workloads import rhs
    torch.cuda.set_device(0)
    rows = []
    cases = [(n, 1e-4) for n in (64, 128, 256, 512)] + [(n, 1e-2) for n in (64, 128, 256)]
    methods = (("dcg", dict(outer="cg")), ("fcg8", dict(outer="fcg", m_max=8)),
               ("fcg8+omg", dict(outer="fcg", m_max=8, outer_mg=args.omg_m, c_A=args.omg_c_A)))
    if args.omg_profile:   # one capped preconditioned solve at the headline size (profiling runs)
        cases, methods = [(args.n, args.dt)], methods[2:]
    elif args.omg_only:    # the preconditioned column only
        methods = methods[2:]
    for n, dt in cases:
        b = torch.from_numpy(rhs(n, 0)).cuda()
        x = torch.empty_like(b)
        for name, kw in methods:
            s = dcg.Solver(n, dt, prec="mixed",
                           max_outer=args.max_outer if args.omg_profile else args.sweep_max_outer,
                           levels=levels_option(n, args.levels), **kw)
            try:
                s.solve(b, x, args.tol)                       # graph capture, caches
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                status, st = s.solve(b, x, args.tol)
                torch.cuda.synchronize()
                t = time.perf_counter() - t0
            except lib.DCGError as e:   # e.g. a breakdown of the outer iteration
                s.close()
                rows.append({"n": n, "dt": dt, "method": name, "status": e.status, "error": str(e)})
                log("omg sweep n=%d dt=%g %s: %s" % (n, dt, name, e))
                continue
            s.close()
            rows.append({"n": n, "dt": dt, "method": name, "status": status, "outer": st.outer_iters,
                         "tot": st.total_wcycles, "solve_s": round(t, 3), "rel_res_true": st.rel_res_true})
            log("omg sweep n=%d dt=%g %s: status %d Out %d Tot %d %.2f s res %.2e"
                % (n, dt, name, status, st.outer_iters, st.total_wcycles, t, st.rel_res_true))
    print(json.dumps({"metric": "outer iterations and solve time against n: DCG, FCG(8), FCG(8) with "
                                "the outer multigrid preconditioner", "m": args.omg_m, "tol": args.tol,
                      "omg_c_A": args.omg_c_A,
                      "rows": rows}), flush=True)


def three_d_table5(args):
    """The analogue of Table 5 (right): deflated CG with the multigrid inner
    solve (W-cycles, RAS, m = 10) at --n3 cubes per side, Out / Tot / Inn for
    dt in {0.5, 0.1, 1e-2, 1e-3, 1e-4} with the fixed rule c_F = 0.01 and the
    adaptive rule c_A = 0.02 and 0.005, tol 1e-8, b = rhs3d(n, 0)."""
    import torch
    import paper_2606_13429_amd as dcg
    from dcg_workloads import THREE_D, rhs3d
    n = args.n3
    torch.cuda.set_device(0)
    b = torch.from_numpy(rhs3d(n, 0)).cuda()
    x = torch.empty_like(b)
    rows = []
    for dt in (0.5, 0.1, 1e-2, 1e-3, 1e-4):
        for rule, c in (("c_F", 0.01), ("c_A", 0.02), ("c_A", 0.005)):
            kw = {"c_F": c} if rule == "c_F" else {"c_A": c}
            s = dcg.Solver3D(n, dt, nu=THREE_D["nu"], penalty=THREE_D["penalty"], inner="mg",
                             max_outer=args.sweep_max_outer, **kw)
            status, st = s.solve(b, x, THREE_D["tol"])
            s.close()
            rows.append({"dt": dt, "rule": rule, "c": c, "status": status, "outer": st.outer_iters,
                         "tot": st.total_wcycles, "inn": round(st.inner_per_outer, 2),
                         "rel_res_true": st.rel_res_true, "ms": round(st.t_solve_ms, 1)})
            log("3d table5 n=%d dt=%g %s=%g: status=%d Out %d Tot %d Inn %.1f res %.2e %.1f ms"
                % (n, dt, rule, c, status, st.outer_iters, st.total_wcycles, st.inner_per_outer,
                   st.rel_res_true, st.t_solve_ms))
    print(json.dumps({"metric": "3D DCG with the multigrid inner solve: Out / Tot / Inn against dt "
                                "and the inner tolerance rule (Table 5, right)", "n": n,
                      "tol": THREE_D["tol"], "rows": rows}), flush=True)


def variants(args):
    """The inner-tolerance rule and outer variant at the headline size: the
    fixed rule (eq. (fixed_tol), c_F = 0.01) against the adaptive rule
    (eq. (tol), c_A = 0.01) with CG, FCG(1), FCG(8) and GMRES; one solve each."""
    import torch
    import paper_2606_13429_amd as dcg
    from dcg_workloads import rhs
    n, dt, tol = args.n, args.dt, args.tol
    torch.cuda.set_device(0)
    b = torch.from_numpy(rhs(n, 0)).cuda()
    x = torch.empty_like(b)
    rows = []
    for outer, c_A in (("cg", 0.0), ("cg", 0.01), ("fcg1", 0.01), ("fcg", 0.01), ("gmres", 0.01)):
        solver = dcg.Solver(n, dt, prec="mixed", outer=outer, c_A=c_A, m_max=8,
                            levels=levels_option(n, args.levels))
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        status, st = solver.solve(b, x, tol)
        torch.cuda.synchronize()
        t = time.perf_counter() - t0
        solver.close()
        rows.append({"outer": outer if outer != "fcg" else "fcg(8)",
                     "inner_rule": "adaptive c_A=0.01" if c_A else "fixed c_F=0.01",
                     "status": status, "outer_iters": st.outer_iters, "tot": st.total_wcycles,
                     "inn": round(st.inner_per_outer, 2), "rel_res_true": st.rel_res_true,
                     "solve_s": round(t, 2)})
        log(str(rows[-1]))
    print(json.dumps({"metric": "inner-tolerance rule / outer variant at n=%d dt=%g, mixed form" % (n, dt),
                      "rows": rows}), flush=True)


def copy_calibration(nbytes):
    """A plain device-to-device copy of ``nbytes`` (torch's copy kernel),
    repeated 5 times: the reference dispatch for scaling HBM traffic counters
    (FETCH_SIZE and WRITE_SIZE should each read nbytes per dispatch)."""
    import torch
    torch.cuda.set_device(0)
    x = torch.ones(nbytes // 8, dtype=torch.float64, device="cuda")
    y = torch.empty_like(x)
    for _ in range(5):
        y.copy_(x)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes": nbytes, "dispatches": 5}), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--n", type=int, default=512)
    ap.add_argument("--dt", type=float, default=1e-4)
    ap.add_argument("--tol", type=float, default=1e-8)
    ap.add_argument("--levels", type=int, default=4,
                    help="multigrid levels of the inner W-cycle (Section 5 uses four; capped at "
                         "the mesh's log2(n/16)+1; 0 = every level down to 16x16 squares)")
    ap.add_argument("--skip-fp64", action="store_true")
    ap.add_argument("--restarts", type=int, default=2,
                    help="warm restarts while the true residual misses tol (0 = the recurrence test only)")
    ap.add_argument("--skip-cpu", action="store_true")
    ap.add_argument("--skip-oracle", action="store_true",
                    help="leave out the comparison with the oracle's golden files")
    ap.add_argument("--max-outer", type=int, default=50000,
                    help="cap on outer iterations (profiling runs only; the headline uses the default)")
    ap.add_argument("--serving", action="store_true",
                    help="run the serving trace instead of the headline solve")
    ap.add_argument("--requests", type=int, default=256, help="serving: trace length")
    ap.add_argument("--serve-max-outer", type=int, default=2000,
                    help="serving: max_outer of every request (NOT_CONVERGED beyond, reported)")
    ap.add_argument("--serve-c-A", type=float, default=0.0,
                    help="serving: adaptive inner tolerance constant (0 = the fixed rule)")
    ap.add_argument("--dt-sweep", action="store_true", help="run the dt sweep at --sweep-n")
    ap.add_argument("--levels-sweep", action="store_true",
                    help="time per W-cycle against the multigrid depth at --n (capped solves)")
    ap.add_argument("--sweep-n", type=int, default=128)
    ap.add_argument("--sweep-max-outer", type=int, default=20000)
    ap.add_argument("--sweep-dts", default="1e-5,1e-4,1e-3,1e-2,1e-1",
                    help="dt sweep: comma-separated time steps")
    ap.add_argument("--sweep-cF", type=float, default=0.01, help="dt sweep: inner tolerance factor")
    ap.add_argument("--sweep-precs", default="fp64,mixed", help="dt sweep: forms to run")
    ap.add_argument("--timestep", action="store_true", help="run BDF2 time stepping at n=1024")
    ap.add_argument("--ts-steps", type=int, default=3)
    ap.add_argument("--ts-outer-mg", type=int, default=0,
                    help="time stepping: FCG(8) with the outer multigrid preconditioner, m steps")
    ap.add_argument("--3d", dest="three_d", action="store_true",
                    help="run the 3D solver at --n3 cubes per side")
    ap.add_argument("--n3", type=int, default=32)
    ap.add_argument("--3d-inner", dest="inner3", choices=("exact", "cg", "mg"), default="exact")
    ap.add_argument("--3d-max-outer", dest="max_outer3", type=int, default=50000,
                    help="3D: cap on outer iterations (profiling runs only)")
    ap.add_argument("--3d-restarts", dest="restarts3", type=int, default=0,
                    help="3D solver: warm restarts while the true residual misses tol")
    ap.add_argument("--3d-levels", dest="levels3", type=int, default=0,
                    help="3D multigrid: levels kept (0 = all, coarsest 2 cubes per side)")
    ap.add_argument("--3d-cA", dest="cA3", type=float, default=0.0,
                    help="3D: adaptive inner tolerance constant (0 = fixed c_F = 0.01)")
    ap.add_argument("--3d-table5", dest="three_d_table5", action="store_true",
                    help="3D multigrid inner solve: Out / Tot / Inn against dt and the inner "
                         "tolerance rule at --n3 (the analogue of Table 5, right)")
    ap.add_argument("--3d-sweep", dest="three_d_sweep", action="store_true",
                    help="outer iterations of the 3D solver against dt at n = 8, 16, 32")
    ap.add_argument("--outer-mg-sweep", action="store_true",
                    help="DCG, FCG(8) and FCG(8) with the outer multigrid preconditioner against n")
    ap.add_argument("--omg-m", type=int, default=4, help="outer multigrid: smoothing steps")
    ap.add_argument("--omg-c-A", dest="omg_c_A", type=float, default=0.0,
                    help="outer multigrid sweep: the adaptive inner tolerance for the preconditioned solves")
    ap.add_argument("--omg-only", action="store_true",
                    help="outer multigrid sweep: the preconditioned solves only")
    ap.add_argument("--omg-profile", action="store_true",
                    help="with --outer-mg-sweep: only the preconditioned solve at --n / --dt, "
                         "capped at --max-outer")
    ap.add_argument("--variants", action="store_true",
                    help="compare the fixed and adaptive inner tolerance at --n/--dt")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="BYTES",
                    help="only run a plain copy of BYTES (traffic-counter calibration)")
    args = ap.parse_args()

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py: this benchmark measures one GPU only; the solve is not sharded across "
              "GPUs (multi-GPU sharding is a design note).  Run with --gpus 1.", file=sys.stderr)
        sys.exit(2)

    if args.copy_calibration:
        copy_calibration(args.copy_calibration)
        return
    if args.serving:
        serving(args)
        return
    if args.variants:
        variants(args)
        return
    if args.levels_sweep:
        levels_sweep(args)
        return
    if args.dt_sweep:
        dt_sweep(args)
        return
    if args.timestep:
        timestep(args)
        return
    if args.three_d:
        three_d(args)
        return
    if args.three_d_sweep:
        three_d_sweep(args)
        return
    if args.three_d_table5:
        three_d_table5(args)
        return
    if args.outer_mg_sweep:
        outer_mg_sweep(args)
        return

    import numpy as np
    import torch
    import paper_2606_13429_amd as dcg
    from paper_2606_13429_amd import _binding as lib
    from dcg_workloads import rhs

    n, dt, tol = args.n, args.dt, args.tol
    torch.cuda.set_device(0)
    J_full = lib.dcg_num_levels(n)
    args.levels = levels_option(n, args.levels)
    levels_in_use = args.levels or J_full
    log("setup n=%d dt=%g (mixed form, %d multigrid levels, <= %d true-residual restarts)"
        % (n, dt, levels_in_use, args.restarts))
    t0 = time.time()
    solver = dcg.Solver(n, dt, prec="mixed", max_outer=args.max_outer, levels=args.levels,
                        restarts=args.restarts)
    log("setup done in %.1f s" % (time.time() - t0))
    bs = [torch.from_numpy(rhs(n, s)).cuda() for s in range(max(args.steps, 1))]
    x = torch.empty_like(bs[0])
    for i in range(args.warmup):
        st = solver.solve(bs[0], x, tol)[1]
        log("warmup %d: outer=%d Tot=%d %.1f ms" % (i, st.outer_iters, st.total_wcycles, st.t_solve_ms))

    lib.dcg_kernel_timing(solver.handle, TIMING_STRIDE)
    stats = []
    x0 = None
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ev0.record()
    for i in range(args.steps):
        status, st = solver.solve(bs[i], x, tol)
        stats.append(dict(st.as_dict(), status_code=status))
        if i == 0:
            x0 = x.clone()        # seed 0's solution, for the same-seed comparisons
        log("step %d: status=%d outer=%d restarts=%d Tot=%d Inn=%.2f res=%.2e %.1f ms"
            % (i, status, st.outer_iters, st.restarts, st.total_wcycles, st.inner_per_outer,
               st.rel_res_true, st.t_solve_ms))
    ev1.record()
    torch.cuda.synchronize()
    ms_total = ev0.elapsed_time(ev1)
    k_ms, k_launches = lib.dcg_kernel_timing_read(solver.handle)
    a_ms, a_launches = lib.dcg_kernel_timing_read_astar(solver.handle)
    lib.dcg_kernel_timing(solver.handle, False)
    ms_per_step = ms_total / args.steps
    value = 1000.0 / ms_per_step

    # dominant kernel: the finest-level RAS step (grouped MFMA kernel).  Its
    # bound is the FP32 matrix pipe: the class inverses come from L2 and its
    # HBM bytes are vectors only; the HBM figures are kept beside.
    k_avg_ms = k_ms / max(k_launches, 1)
    flops = sweep_launch_flops(n)
    tflops = flops / (k_avg_ms * 1e-3) / 1e12
    tiles_bytes = sweep_launch_bytes(n, 4)
    hbm_gbs = tiles_bytes / (k_avg_ms * 1e-3) / 1e9
    cgbs = copy_gbs()
    roofline = {"bound": "mfma", "kernel": "k_sweep_g<float,4> (finest-level RAS step, 4x4 tiles "
                                           "per workgroup, tile solves as FP32 MFMA products)",
                "achieved": round(tflops, 2), "peak": FP32_MFMA_PEAK_TFS, "unit": "TFLOP/s",
                "frac": round(tflops / FP32_MFMA_PEAK_TFS, 4), "traffic": measured_traffic(n),
                "flops_per_launch": flops, "avg_launch_us": round(k_avg_ms * 1e3, 2),
                "launches": k_launches, "timed_every_nth_wcycle": TIMING_STRIDE,
                "hbm_bytes_per_launch": tiles_bytes, "hbm_achieved_gbs": round(hbm_gbs, 1),
                "hbm_frac": round(hbm_gbs / HBM_PEAK_GBS, 4), "copy_gbs": round(cgbs, 1),
                "hbm_frac_of_copy": round(hbm_gbs / cgbs, 4),
                "l2_factor_bytes_per_launch": sweep_l2_factor_bytes(n, 4)}
    if roofline["traffic"]:
        roofline["traffic_over_algorithmic"] = round(roofline["traffic"] / tiles_bytes, 3)
    a_bytes = astar_bytes(n)
    a_avg_ms = a_ms / max(a_launches, 1)
    a_gbs = a_bytes / (a_avg_ms * 1e-3) / 1e9
    roofline_astar = {"bound": "hbm", "kernel": "k_astar (A* product with the direction update)",
                      "achieved": round(a_gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                      "frac": round(a_gbs / HBM_PEAK_GBS, 4), "frac_of_copy": round(a_gbs / cgbs, 4),
                      "avg_launch_us": round(a_avg_ms * 1e3, 2), "launches": a_launches,
                      "bytes_per_launch": a_bytes}

    outer = int(np.mean([s["outer_iters"] for s in stats]))
    nc = n >> (levels_in_use - 1)
    coarse = ("coarsest %dx%d by fast diagonalisation" % (nc, nc) if args.levels
              else "coarsest %dx%d by dense Cholesky" % (nc, nc))
    result = {
        "metric": "dCG solves/s & HBM GB/s, n=512 dt=1e-4, FP32-MG vs FP64; serve p50/p99",
        "value": round(value, 5), "unit": "solves/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(ms_per_step, 2), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f64 outer / f32 multigrid",
        "data": "synthetic: b ~ N(0,1) seeds 0..%d, element-major" % (args.steps - 1),
        "config": {"workload": "deflated CG, unit square %dx%d DG-Q1 (%d dofs), dt=%g, tol=%g on the "
                               "true residual (<= %d warm restarts), W-cycle J=%d (%s) with RAS 4x4+1, "
                               "c_F=0.01, mixed form"
                               % (n, n, 16 * n * n, dt, tol, args.restarts, levels_in_use, coarse),
                   "n": n, "dt": dt, "tol": tol, "form": "mixed", "levels": levels_in_use,
                   "restarts": args.restarts},
        "solve_stats": {"outer_iters": outer,
                        "outer_iters_per_seed": [s["outer_iters"] for s in stats],
                        "restarts_per_seed": [s["restarts"] for s in stats],
                        "total_wcycles": int(np.mean([s["total_wcycles"] for s in stats])),
                        "inner_per_outer": round(float(np.mean([s["inner_per_outer"] for s in stats])), 2),
                        "rel_res_true_max": max(s["rel_res_true"] for s in stats),
                        "converged": sum(s["status_code"] == lib.DCG_OK for s in stats),
                        "setup_ms": round(stats[0]["t_setup_ms"], 1)},
        "roofline": roofline,
        "roofline_astar": roofline_astar,
    }
    if n == 512 and dt == 1e-4 and tol == 1e-8 and levels_in_use == 4 and not args.skip_oracle:
        result["err_vs_oracle"] = err_vs_oracle(dcg)

    if not args.skip_fp64:
        # the all-FP64 form on seed 0, against the mixed form's seed-0 solve
        log("FP64 form: setup + one solve (seed 0)")
        s64 = dcg.Solver(n, dt, prec="fp64", max_outer=args.max_outer, levels=args.levels,
                         restarts=args.restarts)
        x64 = torch.empty_like(x)
        torch.cuda.synchronize()
        t0 = time.time()
        _, st64 = s64.solve(bs[0], x64, tol)
        torch.cuda.synchronize()
        t64 = time.time() - t0
        t_mixed0 = stats[0]["t_solve_ms"] * 1e-3
        result["fp64"] = {"solves_per_s": round(1.0 / t64, 5), "outer_iters": st64.outer_iters,
                          "restarts": st64.restarts, "total_wcycles": st64.total_wcycles,
                          "rel_res_true": st64.rel_res_true,
                          "mixed_speedup_same_seed": round(t64 / t_mixed0, 3),
                          "mixed_vs_fp64_rel_diff": (torch.linalg.norm(x64 - x0)
                                                     / torch.linalg.norm(x64)).item()}
        s64.close()

    if not args.skip_fp64 and args.levels:
        # the same solve on every level down to 16 x 16 squares (dense Cholesky
        # coarsest), for reference
        log("full hierarchy (J=%d): one solve (seed 0)" % J_full)
        sf = dcg.Solver(n, dt, prec="mixed", max_outer=args.max_outer, levels=0,
                        restarts=args.restarts)
        torch.cuda.synchronize()
        t0 = time.time()
        _, stf = sf.solve(bs[0], x, tol)
        torch.cuda.synchronize()
        tf = time.time() - t0
        result["full_hierarchy"] = {"levels": J_full, "solves_per_s": round(1.0 / tf, 5),
                                    "outer_iters": stf.outer_iters, "total_wcycles": stf.total_wcycles,
                                    "rel_res_true": stf.rel_res_true,
                                    "speedup_of_levels_%d_same_seed" % levels_in_use:
                                        round(tf / (stats[0]["t_solve_ms"] * 1e-3), 3)}
        sf.close()

    if not args.skip_fp64:
        # the same seed with a tighter fixed inner tolerance and with the
        # paper's adaptive rule (eq. (tol)); the headline keeps the workload's
        # fixed rule c_F = 0.01
        variants = {}
        for name, kw in (("c_F=1e-4", dict(c_F=1e-4)), ("adaptive c_A=0.01", dict(c_A=0.01))):
            log("inner tolerance %s: one solve (seed 0)" % name)
            sv = dcg.Solver(n, dt, prec="mixed", max_outer=args.max_outer, levels=args.levels,
                            restarts=args.restarts, **kw)
            torch.cuda.synchronize()
            t0 = time.time()
            stv = sv.solve(bs[0], x, tol)[1]
            torch.cuda.synchronize()
            tv = time.time() - t0
            variants[name] = {"solves_per_s": round(1.0 / tv, 5), "outer_iters": stv.outer_iters,
                              "restarts": stv.restarts, "total_wcycles": stv.total_wcycles,
                              "rel_res_true": stv.rel_res_true,
                              "speedup_vs_headline_same_seed":
                                  round(stats[0]["t_solve_ms"] * 1e-3 / tv, 3)}
            sv.close()
        result["inner_tolerance_variants_seed0"] = variants
        # the exact inner solve (fast diagonalisation; the exact-inner deflated CG
        # of Tables 1-2) on the same right-hand side, for reference
        log("exact inner solve: setup + one solve")
        t0 = time.time()
        se = dcg.Solver(n, dt, prec="fp64", inner="exact", max_outer=args.max_outer)
        te_setup = time.time() - t0
        se.solve(bs[0], x, tol)                       # warm-up
        torch.cuda.synchronize()
        t0 = time.time()
        _, ste = se.solve(bs[0], x, tol)
        torch.cuda.synchronize()
        te = time.time() - t0
        result["exact_inner"] = {"solves_per_s": round(1.0 / te, 4), "outer_iters": ste.outer_iters,
                                 "rel_res_true": ste.rel_res_true, "setup_s": round(te_setup, 1),
                                 "ms_per_outer_iteration": round(1e3 * te / max(ste.outer_iters, 1), 3),
                                 "speedup_vs_headline_same_seed":
                                     round(stats[0]["t_solve_ms"] * 1e-3 / te, 2)}
        se.close()
        # the multigrid outer preconditioner (the paper's future work, not its
        # method): FCG(8) with B = one W-cycle on A*, the same right-hand side
        log("outer multigrid preconditioner: setup + one solve")
        t0 = time.time()
        so = dcg.Solver(n, dt, prec="mixed", outer="fcg", m_max=8, outer_mg=args.omg_m,
                        max_outer=args.max_outer, levels=args.levels)
        to_setup = time.time() - t0
        so.solve(bs[0], x, tol)                       # warm-up (graph capture)
        torch.cuda.synchronize()
        t0 = time.time()
        _, sto = so.solve(bs[0], x, tol)
        torch.cuda.synchronize()
        to = time.time() - t0
        result["outer_mg_preconditioner_seed0"] = {
            "method": "FCG(8), directions from B r_i, B = one W-cycle on A* (m = %d), mixed form" % args.omg_m,
            "solves_per_s": round(1.0 / to, 4), "outer_iters": sto.outer_iters,
            "total_wcycles": sto.total_wcycles, "rel_res_true": sto.rel_res_true,
            "setup_s": round(to_setup, 1),
            "speedup_vs_headline_same_seed": round(stats[0]["t_solve_ms"] * 1e-3 / to, 2)}
        so.close()

    if not args.skip_cpu:
        log("CPU oracle baseline (setup is not counted)")
        result["cpu_baseline"] = cpu_baseline(n, dt, tol, outer, result["solve_stats"]["total_wcycles"])
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
