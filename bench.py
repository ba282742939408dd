#!/usr/bin/env python3
"""Benchmark of the RSRR resolvent-sampling hot path on one MI355X.

Workload (default): the dense BEM-like Helmholtz NEP on the unit sphere,
n = 4096 Fibonacci collocation points, ellipse (3.8; 1.4, 0.3), N = 64
sampling points, L = 64 complex Gaussian probes; complex-FP32 LU on the
matrix cores with FP64 iterative refinement.  Inputs are synthetic and
seeded and live in HBM before the timed region starts.

One step = rsrr_sample over all N points (assembly, LU, solves, refinement):
value = N * steps / elapsed (resolvent solves/s).  Unless --sample-only, the
rest of the method (rsrr_basis, rsrr_project, rsrr_solve) then runs once on
the sampled S and its times and eigenvalue diagnostics are reported.

Prints one JSON line (see the repository's benchmark contract), with a
"roofline" object for the LU trailing-update kernel (HIP events around every
launch inside the timed region) and a "cpu_baseline" object (the CPU oracle
timed on a bounded sample of the same workload).
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "resolvent solves/sec (n=4096, L=64) & % MFMA peak; p50/p99 NEP latency"
PEAK_FP32_MFMA_TFLOPS = 157.3
PEAK_FP64_MFMA_TFLOPS = 78.6
PEAK_FP16_MFMA_TFLOPS = 2516.6
# FP32 products as three FP16 products of split operands (the LU's trailing updates of 384 rows and more)
PEAK_SPLIT_TFLOPS = PEAK_FP16_MFMA_TFLOPS / 3
SPLIT_MIN_N = 384
PEAK_HBM_GBS = 8000.0


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="helmholtz", choices=["helmholtz", "delay", "qep", "serve", "batched", "adaptive", "moments", "real",
                                                         "gmres"])
    ap.add_argument("--n", type=int, default=None)
    ap.add_argument("--N", type=int, default=None)
    ap.add_argument("--L", type=int, default=None)
    ap.add_argument("--prec", default="mixed", choices=["mixed", "c128"])
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--cpu-points", type=int, default=None, help="sampling points in the CPU sample")
    ap.add_argument("--no-plain", action="store_true",
                    help="skip the comparison run (plain FP64 sampling; for gmres the direct path)")
    ap.add_argument("--sample-only", action="store_true", help="skip the basis/projection/SS-FULL pass")
    ap.add_argument("--nq", type=int, default=500, help="SS-FULL quadrature nodes")
    ap.add_argument("--latency-runs", type=int, default=5, help="whole-method runs for the NEP latency p50/p99")
    ap.add_argument("--calib-copy", action="store_true",
                    help="run one plain 1 GiB device copy before the timed region (counter calibration)")
    ap.add_argument("--instances", type=int, default=256, help="batched: QEP instances")
    ap.add_argument("--n1", type=int, default=6, help="adaptive: stage-1 contour points")
    ap.add_argument("--K", type=str, default="4,16", help="moments: moment counts K to compare")
    ap.add_argument("--real-nep", default="delay", choices=["delay", "string"], help="real: the real NEP")
    ap.add_argument("--interval", type=str, default=None, help="real: sampling interval lo,hi")
    ap.add_argument("--gmres-nep", default="helmholtz", choices=["helmholtz", "delay", "sparse"],
                    help="gmres: the NEP (sparse: the delay Laplacian on a 3D grid, matrices in CSR)")
    ap.add_argument("--nref", type=int, default=1, help="gmres: reference points (factorisations)")
    ap.add_argument("--restart", type=int, default=32, help="gmres: restart cycle length")
    ap.add_argument("--tol", type=float, default=1e-10, help="gmres: relative residual per column")
    ap.add_argument("--requests", type=int, default=24, help="serve: requests taken from the stream")
    ap.add_argument("--rate", type=float, default=20.0, help="serve: Poisson arrival rate (1/s)")
    ap.add_argument("--slots", type=int, default=8, help="serve: requests admitted at once")
    ap.add_argument("--arena-gb", type=int, default=150,
                    help="serve: HBM arena for the requests' footprints (S, kept factors, Q, V) (GiB)")
    ap.add_argument("--batch-gb", type=int, default=48, help="serve: LU workspace cap per launch (GiB)")
    ap.add_argument("--solvers", type=int, default=0, help="serve: solve threads (0: library default)")
    ap.add_argument("--serve-leg", type=int, default=24,
                    help="default workload: requests of the serving leg run after the headline (0: none)")
    ap.add_argument("--serve-slow-rate", type=float, default=1.5,
                    help="default workload: the serving leg's second, sustainable arrival rate (1/s)")
    return ap.parse_args()


def build_workload(args):
    import workloads as W
    if args.workload == "helmholtz":
        n = args.n or 4096
        nep, C, U = W.cfg_helmholtz(n=n, N=args.N or 64, L=args.L or 64)
        desc = f"helmholtz_sphere n={n} N={C.N} L={U.shape[1]} ellipse(3.8;1.4,0.3)"
    elif args.workload == "delay":
        nx = int(round(math.sqrt(args.n or 1024)))
        nep, C, U = W.cfg_delay(nx=nx, N=args.N or 48, L=args.L or 32, parity=False)
        desc = f"delay_laplacian n={nep.n} N={C.N} L={U.shape[1]} circle(-20,15)"
    else:
        nep, C, U = W.cfg_qep(n=args.n or 200, N=args.N or 32, L=args.L or 16)
        desc = f"rotated_diag_qep n={nep.n} N={C.N} L={U.shape[1]} ellipse(5i;4,1)"
    return nep, C, U, desc


def _profile_figure(name, key, conv):
    """A figure from a committed rocprofv3 counter summary under profiles/, or None when the
    kernels or the LU driver have changed since the counters were taken (hash of the files)."""
    import hashlib
    path = os.path.join(ROOT, "profiles", name)
    srcs = [os.path.join(ROOT, "paper_1605_07951_amd", "csrc", f) for f in ("gemm.hip", "lu.hip", "split.hip")]
    try:
        txt = open(path).read()
        val = conv(txt.split(key + ":")[1].split()[0])
        sha = txt.split("source_sha256_16 (csrc/gemm.hip + csrc/lu.hip + csrc/split.hip):")[1].split()[0]
        h = hashlib.sha256(b"".join(open(s, "rb").read() for s in srcs)).hexdigest()[:16]
    except (OSError, IndexError, ValueError):
        return None
    return val if h == sha else None


def measured_traffic():
    """HBM bytes per trailing-update launch (FETCH_SIZE + WRITE_SIZE, copy-calibrated)."""
    return _profile_figure("traffic_trailing_update_helmholtz_n4096_N64_L64_mixed.md",
                           "traffic_bytes_per_launch", int)


def measured_mfma_util():
    """rocprofv3's MfmaUtil of the trailing update (mean over one step's launches)."""
    return _profile_figure("mfma_util_trailing_update_helmholtz_n4096_N64_L64_mixed.md",
                           "rocprof_mfma_util_update", float)


def phase_rooflines(n, N, L, tm, iters):
    """Achieved rates of the sampling phases other than the LU, from the last step's phase times.

    Work per step (all N points are processed by every launch of a pass, converged points
    included): the Helmholtz assembly writes a c64 copy of T for the LU and a c128 copy for the
    residual (24 n^2 bytes per point; the entries are generated, nothing n^2-sized is read);
    the solve and the FP64 residual each run once before refinement and once per correction
    (iters + 1 passes).  A solve pass reads the c64 factors (8 n^2 bytes) and does 8 n^2 L
    flops (standard complex count) per point; a residual pass reads T in c128 (16 n^2 bytes)
    and does 8 n^2 L FP64 flops per point.  With L = 64 both passes sit above the ridge of
    their matrix peak (8 L flops per 8-byte factor entry against 157.3 / 8 = 19.7; 8 L per
    16-byte entry against 78.6 / 8 = 9.8), so their flop rate is the one that bounds them."""
    n2 = float(n) * n
    passes = iters + 1
    out = {}
    a_ms = tm.get("assemble_ms", 0.0)
    if a_ms > 0:
        b = N * 24.0 * n2
        out["assembly"] = {"ms": round(a_ms, 3), "bytes": b, "GB_s": round(b / (a_ms * 1e-3) / 1e9, 1),
                           "hbm_frac": round(b / (a_ms * 1e-3) / 1e9 / PEAK_HBM_GBS, 4)}
    s_ms = tm.get("solve_ms", 0.0)
    if s_ms > 0:
        f = passes * N * 8.0 * n2 * L
        b = passes * N * 8.0 * n2
        out["solves"] = {"ms": round(s_ms, 3), "passes": passes, "flops": f, "bytes": b,
                         "TFLOP_s": round(f / (s_ms * 1e-3) / 1e12, 2),
                         "fp32_mfma_frac": round(f / (s_ms * 1e-3) / 1e12 / PEAK_FP32_MFMA_TFLOPS, 4),
                         "GB_s": round(b / (s_ms * 1e-3) / 1e9, 1)}
    r_ms = tm.get("residual_ms", 0.0)
    if r_ms > 0:
        f = passes * N * 8.0 * n2 * L
        b = passes * N * 16.0 * n2
        out["residual"] = {"ms": round(r_ms, 3), "passes": passes, "flops": f, "bytes": b,
                           "TFLOP_s": round(f / (r_ms * 1e-3) / 1e12, 2),
                           "fp64_mfma_frac": round(f / (r_ms * 1e-3) / 1e12 / PEAK_FP64_MFMA_TFLOPS, 4),
                           "GB_s": round(b / (r_ms * 1e-3) / 1e9, 1)}
    return out


def cpu_model():
    """CPU model name and logical CPUs this process may run on (Linux)."""
    model = None
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    try:
        avail = len(os.sched_getaffinity(0))
    except AttributeError:
        avail = os.cpu_count() or 1
    return model, avail


def cpu_baseline(nep, C, U, npts):
    """Time the CPU oracle's sampling on npts points of the same workload.  `cores` is the
    BLAS thread count the oracle's LAPACK calls ran with (threadpoolctl), never more than the
    CPUs available to the process."""
    from oracle import rsrr_oracle as O
    model, avail = cpu_model()
    threads = avail
    blas = None
    try:
        from threadpoolctl import threadpool_info
        info = [i for i in threadpool_info() if i.get("user_api") == "blas"] or threadpool_info()
        if info:
            threads = min(avail, max(int(i.get("num_threads", 1)) for i in info))
            blas = f"{info[0].get('internal_api')} {info[0].get('version')}"
    except Exception:
        pass
    prob = O.Problem(nep)
    z, _ = O.ellipse(C.gamma, C.a, C.b, C.N)
    pts = z[:npts]
    t0 = time.perf_counter()
    O.sample(prob, pts, U)
    dt = time.perf_counter() - t0
    return {"value": npts / dt, "unit": "resolvent solves/s", "cores": threads, "kind": "oracle",
            "cpu_model": model, "cpus_available": avail, "blas": blas,
            "sample": f"{npts} of {C.N} sampling points of the same workload (assembly + zgetrf + zgetrs, "
                      f"FP64, NumPy/SciPy LAPACK), {dt:.2f} s"}



def _pct(x, q):
    return float(np.percentile(np.asarray(x), q)) if len(x) else None


def serving_items(requests, rate):
    """The first `requests` entries of the seeded serving stream with their device inputs: one
    DeviceNEP per (kind, n) (the NEP depends only on those), probes per request."""
    import torch
    import workloads as W
    from paper_1605_07951_amd import rsrr as R

    stream = W.cfg_serving_stream(count=requests, rate=rate)
    neps, items = {}, []
    for q in stream:
        key = (q["kind"], q["n"])
        if key not in neps:
            neps[key] = R.DeviceNEP(W.serving_nep(q))
        items.append((q, neps[key], R.colmajor(W.probes(q["n"], q["L"], q["seed"]))[0]))
    torch.cuda.synchronize()
    return items


def serve_stream(items, label, prec, flags, slots, arena_gb, batch_gb, solvers=0, rate_scale=1.0):
    """Submit the items at their arrival times (scaled by rate_scale: times are divided by it)
    to a fresh server and wait for all; latency = result on the host minus submission."""
    import threading
    from paper_1605_07951_amd import rsrr as R

    srv = R.Server(prec=prec, max_slots=slots, arena_bytes=arena_gb << 30, batch_bytes=batch_gb << 30,
                   flags=flags, solvers=solvers)
    ids = [None] * len(items)
    t0 = time.perf_counter()

    def feeder():
        for i, (q, dn, U) in enumerate(items):
            dt = q["t"] / rate_scale - (time.perf_counter() - t0)
            if dt > 0:
                time.sleep(dt)
            ids[i] = srv.submit(dn, U, q["gamma"], q["a"], q["b"], q["N"], max_eigs=64)

    th = threading.Thread(target=feeder)
    th.start()
    th.join()
    res = []
    for i in range(len(items)):
        res.append(srv.wait(ids[i]))
        r = res[-1]
        print(f"[serve {label}] {i + 1}/{len(items)} {items[i][0]['kind']} n={items[i][0]['n']} "
              f"latency {r['t_done'] - r['t_submit']:.3f}s status {r['status']}", file=sys.stderr, flush=True)
    elapsed = time.perf_counter() - t0
    st = srv.stats()
    srv.close()
    lat = [r["t_done"] - r["t_submit"] for r in res]
    t_first = min(r["t_submit"] for r in res)
    makespan = max(r["t_done"] for r in res) - t_first
    solves = sum(q["N"] for q, _, _ in items)
    worst, n_inside = 0.0, 0
    for (q, _, _), r in zip(items, res):
        d = r["lam"] - complex(q["gamma"])
        ins = (d.real / q["a"]) ** 2 + (d.imag / q["b"]) ** 2 < 0.98
        n_inside += int(ins.sum())
        if ins.any():
            worst = max(worst, float(r["resid"][ins].max()))
    span = items[-1][0]["t"] / rate_scale
    out = {"requests": len(items), "offered_rate_per_s": round(len(items) / span, 3) if span > 0 else None,
           "p50_latency_s": round(_pct(lat, 50), 4), "p99_latency_s": round(_pct(lat, 99), 4),
           "mean_latency_s": round(float(np.mean(lat)), 4), "makespan_s": round(makespan, 3),
           "mean_wait_admit_s": round(float(np.mean([r["t_admit"] - r["t_submit"] for r in res])), 4),
           "mean_sampling_s": round(float(np.mean([r["t_sampled"] - r["t_admit"] for r in res])), 4),
           "mean_post_s": round(float(np.mean([r["t_done"] - r["t_sampled"] for r in res])), 4),
           "req_per_s": round(len(items) / makespan, 3), "solves_per_s": round(solves / makespan, 3),
           "wall_s": round(elapsed, 3), "launches": int(st["launches"]),
           "max_launch_points": int(st["max_launch_points"]), "sampler_busy_s": round(st["sampler_busy_s"], 3),
           "solver_busy_s": round(st["solver_busy_s"], 3), "arena_peak_gb": round(st["arena_peak_bytes"] / 2**30, 3),
           "device_mem_peak_gb": round(st["device_mem_peak_bytes"] / 2**30, 2),
           "statuses": {str(k): int(v) for k, v in zip(*np.unique([r["status"] for r in res], return_counts=True))},
           "eigs_inside": n_inside, "reprobes": int(st["reprobes"]),
           "eig_resid_max_inside": worst, "fallback_points": int(sum(r["fallbacks"] for r in res))}
    return out, solves


def run_serve(args):
    """Serving stream: requests arrive (Poisson), the server batches their sampling points.

    Latency = result on the host minus submission (at the arrival time).  The
    same stream is then replayed through a sequential plain-FP64 server (one
    slot, no batching, no overlap) for comparison."""
    from paper_1605_07951_amd import rsrr as R

    items = serving_items(args.requests, args.rate)
    print(f"[serve] {len(items)} requests ready", file=sys.stderr, flush=True)
    served, solves = serve_stream(items, "mixed", R.RSRR_PREC_C64_IR, 0, args.slots, args.arena_gb, args.batch_gb,
                                  args.solvers)
    res = {
        "metric": METRIC,
        "value": served["solves_per_s"],
        "unit": "resolvent solves/s",
        "n_gpus": 1,
        "steps": len(items),
        "warmup": 0,
        "ms_per_step": round(1e3 * served["makespan_s"] / len(items), 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c64 LU (f32 panels and sums, split-f16 MFMA updates) + f64 refinement",
        "data": "synthetic (seeded serving stream: delay Laplacian and Helmholtz sphere NEPs, Gaussian probes)",
        "config": {"workload": f"serving stream: first {len(items)} of the seeded 2000-request stream, Poisson "
                               f"{args.rate}/s, 50/50 delay (n 512/1024/2048, N=48, L=32) / Helmholtz "
                               f"(n 2048/4096/8192, N=64, L=64)",
                   "slots": args.slots, "arena_gb": args.arena_gb, "batch_gb": args.batch_gb,
                   "step": "one request: contour, sampling, basis, projection, SS-FULL, eigenpairs on the host"},
        "roofline": None,
        "serving": served,
    }
    if not args.no_plain:
        seq, _ = serve_stream(items, "fp64-seq", R.RSRR_PREC_C128, R.RSRR_SERVE_NO_BATCH | R.RSRR_SERVE_SERIAL, 1,
                              args.arena_gb, args.batch_gb)
        res["sequential_plain_fp64"] = seq
        res["speedup_vs_sequential_fp64"] = {
            "solves_per_s": round(served["solves_per_s"] / seq["solves_per_s"], 3),
            "p50_latency": round(seq["p50_latency_s"] / served["p50_latency_s"], 3),
            "p99_latency": round(seq["p99_latency_s"] / served["p99_latency_s"], 3)}
    print(json.dumps(res), flush=True)


def run_batched(args):
    """Ragged batch: QEP instances with n ~ U{64..1024}, N=24, L=8 each, ellipse (5i; 4, 1).

    Step = every sampling point of every instance through rsrr_sample_batched
    (size buckets, device-side refinement).  value = points / step time with
    the bucket work captured once in hipGraphs and replayed; the eager batched
    call and a loop of one rsrr_sample call per instance are timed beside it."""
    import torch
    import workloads as W
    from paper_1605_07951_amd import rsrr as R

    sizes = [int(n) for n in W.cfg_batched_sizes(count=args.instances)]
    N, L = 24, 8
    z, _ = R.rsrr_contour(5j, 4.0, 1.0, N)
    items = [R.BatchItem(R.DeviceNEP(W.rotated_diagonal_qep(n, 3000 + i)), z, W.probes(n, L, 30000 + i))
             for i, n in enumerate(sizes)]
    ctx = R.rsrr_create(0)
    solves = len(sizes) * N
    lu_flops = sum(8.0 / 3.0 * n ** 3 for n in sizes) * N
    torch.cuda.synchronize()
    print(f"[batched] {len(items)} instances ready", file=sys.stderr, flush=True)

    def timed(fn, steps, warmup):
        for _ in range(warmup):
            fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            out = fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / steps, out

    t0 = time.perf_counter()
    R.rsrr_sample_batched(ctx, items, flags=R.RSRR_BATCH_AUTOTUNE)
    torch.cuda.synchronize()
    tune_s = time.perf_counter() - t0
    eager_s, _ = timed(lambda: R.rsrr_sample_batched(ctx, items, flags=0), args.steps, args.warmup)
    t0 = time.perf_counter()
    R.rsrr_sample_batched(ctx, items, flags=R.RSRR_BATCH_GRAPH)  # capture
    torch.cuda.synchronize()
    capture_s = time.perf_counter() - t0
    graph_s, (infos, _) = timed(lambda: R.rsrr_sample_batched(ctx, items, flags=R.RSRR_BATCH_GRAPH),
                                args.steps, args.warmup)

    def loop():
        for it in items:
            R.rsrr_sample(ctx, it.dnep, z, it.U, S=it.S)
    loop_s, _ = timed(loop, 1, 1)
    resid = max(max(p["resid"] for p in inf) for inf in infos)
    fb = sum(sum(p["fallback"] for p in inf) for inf in infos)
    iters_hist = np.bincount([p["ir_iters"] for inf in infos for p in inf]).tolist()
    achieved = lu_flops / graph_s / 1e12
    res = {
        "metric": METRIC,
        "value": round(solves / graph_s, 3),
        "unit": "resolvent solves/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(1e3 * graph_s, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c64 LU (f32 panels and sums, split-f16 MFMA updates) + f64 refinement",
        "data": "synthetic (seeded rotated diagonal QEPs, complex Gaussian probes)",
        "config": {"workload": f"ragged batch: {len(sizes)} rotated diagonal QEPs, n ~ U{{64..1024}} "
                               f"(sum n = {sum(sizes)}), N={N}, L={L}, ellipse (5i; 4, 1)",
                   "step": "all points of all instances: assembly, LU, solves, refinement (hipGraph replay)"},
        # buckets of 384 rows and more update with split FP16 operands, smaller ones in FP32
        "roofline": {"bound": "mfma", "kernel": "whole batched step (LU algorithmic flops / step time)",
                     "achieved": round(achieved, 3), "peak": round(PEAK_SPLIT_TFLOPS, 1), "unit": "TFLOP/s",
                     "frac": round(achieved / PEAK_SPLIT_TFLOPS, 4), "traffic": None},
        "batched": {"graph_ms": round(1e3 * graph_s, 3), "eager_ms": round(1e3 * eager_s, 3),
                    "per_instance_loop_ms": round(1e3 * loop_s, 3), "capture_ms": round(1e3 * capture_s, 1),
                    "autotune_first_call_ms": round(1e3 * tune_s, 1),
                    "graph_over_loop_speedup": round(loop_s / graph_s, 3),
                    "graph_over_eager_speedup": round(eager_s / graph_s, 3),
                    "resid_max": resid, "fallbacks": fb, "ir_iters_histogram": iters_hist,
                    "lu_tflop_per_step": round(lu_flops / 1e12, 4)},
    }
    print(json.dumps(res), flush=True)


def run_adaptive(args):
    """Two-stage sampling on the Helmholtz sphere (n=4096, L=16, ellipse (3.8; 1.4, 0.3)):
    stage 1 on --n1 contour points, stage 2 adds the estimates inside as points.  Timed
    beside the one-stage method on the 64-point contour (same L)."""
    import torch
    import workloads as W
    from paper_1605_07951_amd import rsrr as R

    n = args.n or 4096
    nep, C, U_host = W.cfg_helmholtz(n=n, N=64, L=args.L or 16)
    dnep = R.DeviceNEP(nep)
    U, _ = R.colmajor(U_host)
    ctx = R.rsrr_create(0)
    R.rsrr_two_stage(ctx, dnep, C.gamma, C.a, C.b, args.n1, U, max_new=16, max_eigs=64)  # warm-up
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    two = R.rsrr_two_stage(ctx, dnep, C.gamma, C.a, C.b, args.n1, U, max_new=16, max_eigs=64)
    torch.cuda.synchronize()
    t_two = time.perf_counter() - t0

    def inside(lam):
        d = lam - complex(C.gamma)
        return (d.real / C.a) ** 2 + (d.imag / C.b) ** 2 < 1

    t0 = time.perf_counter()
    z, _ = R.rsrr_contour(C.gamma, C.a, C.b, 64)
    S, _, _ = R.rsrr_sample(ctx, dnep, z, U)
    Q, k, _ = R.rsrr_basis(ctx, S, n, 1e-14)
    AQ, terms = R.rsrr_project(ctx, dnep, Q, k, C.gamma, max(C.a, C.b))
    one = R.rsrr_solve(ctx, dnep, Q, k, AQ, terms, C.gamma, C.a, C.b)
    torch.cuda.synchronize()
    t_one = time.perf_counter() - t0
    i2, i1 = inside(two["lam"]), inside(one["lam"])
    pts = args.n1 + two["n_new"]
    res = {
        "metric": METRIC,
        "value": round(pts / t_two, 3),
        "unit": "resolvent solves/s",
        "n_gpus": 1, "steps": 1, "warmup": 1, "ms_per_step": round(1e3 * t_two, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "c64 LU (f32 panels and sums, split-f16 MFMA updates) + f64 refinement",
        "data": "synthetic (seeded Fibonacci-sphere Helmholtz single-layer NEP, complex Gaussian probes)",
        "config": {"workload": f"two-stage sampling, helmholtz_sphere n={n} L={U_host.shape[1]} "
                               f"ellipse(3.8;1.4,0.3), stage 1 on {args.n1} contour points",
                   "step": "whole two-stage method (both stages: sampling, basis, projection, SS-FULL)"},
        "roofline": None,
        "two_stage": {"points": pts, "n_new": two["n_new"], "k1": two["k1"], "k2": two["k2"],
                      "stage1_resid_max_inside": two["resid1_max"],
                      "stage2_eigs_inside": int(i2.sum()),
                      "stage2_resid_max_inside": float(two["resid"][i2].max()) if i2.any() else None,
                      "seconds": round(t_two, 3),
                      "lambda_inside": [[float(l.real), float(l.imag)] for l in two["lam"][i2]]},
        "one_stage_64_points": {"eigs_inside": int(i1.sum()),
                                "resid_max_inside": float(one["resid"][i1].max()) if i1.any() else None,
                                "seconds": round(t_one, 3)},
    }
    print(json.dumps(res), flush=True)


def run_moments(args):
    """Sampling scheme vs moment scheme on the same S (Helmholtz sphere n=4096, N=64, L=64):
    M = S Z for several K, then Steps 3-5 on S and on each M; reports the rank kept, the
    eigen-residuals inside the contour and the time of M = S Z (one batched FP64 GEMM)."""
    import torch
    import workloads as W
    from paper_1605_07951_amd import rsrr as R

    n = args.n or 4096
    nep, C, U_host = W.cfg_helmholtz(n=n, N=args.N or 64, L=args.L or 64)
    dnep = R.DeviceNEP(nep)
    U, _ = R.colmajor(U_host)
    L, N = U_host.shape[1], C.N
    ctx = R.rsrr_create(0)
    z, _ = R.rsrr_contour(C.gamma, C.a, C.b, N)
    S, _, _ = R.rsrr_sample(ctx, dnep, z, U)
    rho = max(C.a, C.b)
    cap = (C.a + C.b) / (2 * rho)

    def steps(X):
        t0 = time.perf_counter()
        Q, k, sig = R.rsrr_basis(ctx, X.clone(), n, 1e-14)
        AQ, terms = R.rsrr_project(ctx, dnep, Q, k, C.gamma, rho)
        out = R.rsrr_solve(ctx, dnep, Q, k, AQ, terms, C.gamma, C.a, C.b)
        torch.cuda.synchronize()
        d = out["lam"] - complex(C.gamma)
        ins = (d.real / C.a) ** 2 + (d.imag / C.b) ** 2 < 1
        return {"k": k, "eigs_inside": int(ins.sum()),
                "resid_max_inside": float(out["resid"][ins].max()) if ins.any() else None,
                "sigma_ratio_at_64": float(sig[min(63, sig.size - 1)] / sig[0]),
                "steps_3_5_s": round(time.perf_counter() - t0, 3)}

    res_s = steps(S)
    rows = {}
    for K in [int(x) for x in args.K.split(",")]:
        K = min(K, N)
        R.rsrr_moments(ctx, S, n, z, L, K, C.gamma, rho, cap)  # warm-up
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        M = R.rsrr_moments(ctx, S, n, z, L, K, C.gamma, rho, cap)
        torch.cuda.synchronize()
        tm = time.perf_counter() - t0
        r = steps(M)
        r["moments_ms"] = round(1e3 * tm, 3)
        r["moments_tflops"] = round(8.0 * n * N * K * L / tm / 1e12, 3)
        rows[f"K={K}"] = r
    res = {
        "metric": METRIC, "value": None, "unit": "resolvent solves/s", "n_gpus": 1, "steps": 1, "warmup": 1,
        "ms_per_step": None, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f64", "data": "synthetic (seeded Fibonacci-sphere Helmholtz single-layer NEP, complex Gaussian probes)",
        "config": {"workload": f"sampling vs moment scheme on one S: helmholtz_sphere n={n} N={N} L={L}",
                   "step": "M = S Z and Steps 3-5 on S and on M"},
        "roofline": None,
        "sampling_scheme": res_s,
        "moment_scheme": rows,
    }
    print(json.dumps(res), flush=True)


def run_real(args):
    """Real sampling of a real NEP at N Chebyshev points of a real interval, L real probes.
    Default: the delay Laplacian on a 64x64 grid (n=4096), interval [-9, -4] (it holds real
    eigenvalues), N=64, L=16; --real-nep string: the loaded string of Example 1 on [3, 10000].
    value = resolvent solves/s of the real FP32 LU path (R32_IR); the complex FP32 and FP64
    paths run on the same inputs."""
    import torch
    import workloads as W
    from paper_1605_07951_amd import rsrr as R

    N = args.N or 64
    L = args.L or 16
    if args.real_nep == "string":
        n = args.n or 4096
        nep = W.loaded_string(n)
        lo, hi = 3.0, 10000.0
    else:
        nx = int(round(math.sqrt(args.n or 4096)))
        nep = W.delay_laplacian(nx)
        n = nep.n
        lo, hi = -9.0, -4.0
    if args.interval:
        lo, hi = (float(v) for v in args.interval.split(","))
    dnep = R.DeviceNEP(nep)
    z = W.interval_points(lo, hi, N)
    U, _ = R.colmajor(W.real_probes(n, L, 78))
    ctx = R.rsrr_create(0)
    S = torch.empty((N * L, n), dtype=torch.complex128, device="cuda")
    out = {}
    for name, prec in (("r32", R.RSRR_PREC_R32_IR), ("c64", R.RSRR_PREC_C64_IR), ("c128", R.RSRR_PREC_C128)):
        for _ in range(args.warmup):
            R.rsrr_sample(ctx, dnep, z, U, prec=prec, S=S)
        torch.cuda.synchronize()
        R.rsrr_update_stats(ctx, enable=True, reset=True)
        t0 = time.perf_counter()
        for _ in range(args.steps):
            _, info, _ = R.rsrr_sample(ctx, dnep, z, U, prec=prec, S=S)
        torch.cuda.synchronize()
        dt = (time.perf_counter() - t0) / args.steps
        st = R.rsrr_update_stats(ctx, enable=False)
        out[name] = {"solves_per_s": round(N / dt, 3), "ms_per_step": round(1e3 * dt, 3),
                     "update_tflops": round(st["flops"] / (st["ms"] * 1e-3) / 1e12, 3) if st["ms"] > 0 else None,
                     "update_launches": st["launches"],
                     "resid_max": max(i["resid"] for i in info), "fallbacks": sum(i["fallback"] for i in info),
                     "ir_iters_max": max(i["ir_iters"] for i in info)}
    r32 = out["r32"]
    achieved = r32["update_tflops"] or 0.0
    split = n >= SPLIT_MIN_N
    peak = PEAK_SPLIT_TFLOPS if split else PEAK_FP32_MFMA_TFLOPS
    res = {
        "metric": METRIC,
        "value": r32["solves_per_s"],
        "unit": "resolvent solves/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": r32["ms_per_step"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32 LU (f32 panels and sums, split-f16 MFMA updates) + f64 refinement",
        "data": f"synthetic ({nep.name}, real Gaussian probes)",
        "config": {"workload": f"real sampling, {nep.name} n={n}, N={N} Chebyshev points of [{lo}, {hi}], L={L}",
                   "step": "rsrr_sample over all N points (assembly, real LU, solves, refinement)"},
        "roofline": {"bound": "mfma", "kernel": "LU trailing update, real "
                     + ("(gemm_split_kernel<float,true>)" if split else "(sgemm_mfma_kernel<*,1>)"),
                     "achieved": achieved, "peak": round(peak, 1), "unit": "TFLOP/s",
                     "frac": round(achieved / peak, 4), "traffic": None},
        "paths": out,
        "r32_over_c64": round(out["r32"]["solves_per_s"] / out["c64"]["solves_per_s"], 3),
        "r32_over_c128": round(out["r32"]["solves_per_s"] / out["c128"]["solves_per_s"], 3),
    }
    print(json.dumps(res), flush=True)

def run_gmres(args):
    """Iterative sampling: flexible GMRES per column, preconditioned by complex FP32 LU factors of T
    at --nref reference points (one factorisation serves many points), FP64 operator and residuals.
    Default: the Helmholtz sphere NEP (n=4096) on the headline ellipse with N=64 points and L=2
    probes (the probe count of the paper's large boundary-element runs), one reference at the
    contour centre, tol 1e-10.  --gmres-nep delay: the delay Laplacian (64x64 grid) on its
    parity circle (centre -4, radius 0.75).  --gmres-nep sparse: the delay Laplacian on a 3D grid
    (20^3, n = 8000) with its matrices in CSR, the operator applied from the sparse rows; the same
    NEP with dense matrices (the dense separable operator) runs beside it.  The direct
    mixed-precision path runs on the same inputs for comparison.
    value = resolvent solves/s (points per second) of the GMRES path."""
    import torch
    import workloads as W
    from paper_1605_07951_amd import rsrr as R

    N = args.N or 64
    L = args.L or 2
    n = args.n or 4096
    if args.gmres_nep == "helmholtz":
        nep, C, Uh = W.cfg_helmholtz(n=n, N=N, L=L)
    elif args.gmres_nep == "sparse":
        side = int(round((args.n or 8000) ** (1.0 / 3.0)))
        nep, C, Uh = W.cfg_sparse(dims=(side, side, side), N=N, L=L)
        n = nep.n
    else:
        nep, C, Uh = W.cfg_delay(nx=int(round(math.sqrt(n))), N=N, L=L)
        n = nep.n
    dnep = R.DeviceNEP(nep)
    z, _ = R.rsrr_contour(C.gamma, C.a, C.b, C.N)
    zref = [C.gamma] if args.nref == 1 else R.rsrr_contour(C.gamma, 0.5 * C.a, 0.5 * C.b, args.nref)[0]
    U, _ = R.colmajor(Uh)
    ctx = R.rsrr_create(0)
    S = torch.empty((N * L, n), dtype=torch.complex128, device="cuda")

    def gm():
        return R.rsrr_sample_gmres(ctx, dnep, z, U, zref, tol=args.tol, restart=args.restart, S=S)

    for _ in range(args.warmup):
        gm()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        _, info, _ = gm()
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / args.steps
    tm = ctx.raw_timings()
    iters = [i["iters"] for i in info]
    cycles = max(i["restarts"] for i in info) + 1
    applies = max(iters) + cycles           # Arnoldi steps in lockstep + one true residual per cycle
    op_ms = tm[1] / applies
    sparse = hasattr(nep, "csr")
    if sparse:
        # each apply reads every term's rows once (row pointers, columns, values) and the n x N L
        # block in, and writes the block out
        csr_bytes = sum(4.0 * ip.size + 20.0 * ix.size for ip, ix, _ in nep.csr)
        bytes_apply = csr_bytes + 2 * 16.0 * n * N * L
        achieved = bytes_apply / (op_ms * 1e-3) / 1e9
        roof = {"bound": "hbm", "kernel": "operator sum_j f_j A_j Z from the sparse rows, FP64 (csr_apply_kernel)",
                "achieved": round(achieved, 1), "peak": 8000.0, "unit": "GB/s",
                "frac": round(achieved / 8000.0, 4), "traffic": None,
                "bytes_per_apply": bytes_apply, "avg_apply_ms": round(op_ms, 4), "applies": applies,
                "nnz": int(sum(ix.size for _, ix, _ in nep.csr))}
    elif not hasattr(nep, "A") and info[0]["matrix_free"]:
        # entries generated inside every application: transcendental FP64 work, no stored matrices
        roof = None
    elif not hasattr(nep, "A"):
        # each apply streams the N assembled FP64 matrices once (plus the n x L blocks in and out)
        bytes_apply = N * 16.0 * n * n + 2 * 16.0 * n * N * L
        achieved = bytes_apply / (op_ms * 1e-3) / 1e9
        roof = {"bound": "hbm", "kernel": "operator T(z_k) Z, FP64 (resid_stream_kernel, R = T X form)",
                "achieved": round(achieved, 1), "peak": 8000.0, "unit": "GB/s",
                "frac": round(achieved / 8000.0, 4), "traffic": None,
                "bytes_per_apply": bytes_apply, "avg_apply_ms": round(op_ms, 4), "applies": applies}
    else:
        J = len(nep.A)
        flops_apply = J * 8.0 * n * n * N * L
        achieved = flops_apply / (op_ms * 1e-3) / 1e12
        roof = {"bound": "mfma", "kernel": "operator sum_j A_j (Z f_j), FP64 (zgemm_mfma_kernel)",
                "achieved": round(achieved, 3), "peak": PEAK_FP64_MFMA_TFLOPS, "unit": "TFLOP/s",
                "frac": round(achieved / PEAK_FP64_MFMA_TFLOPS, 4), "traffic": None,
                "flops_per_apply": flops_apply, "avg_apply_ms": round(op_ms, 4), "applies": applies}
    mfree = None
    dense_op = None
    if sparse and not args.no_plain:
        # the same NEP with its matrices stored densely: the dense separable operator
        from scipy import sparse as sps
        dn = R.DeviceNEP(W.SeparableNEP(nep.name + "_dense",
                                        [sps.csr_matrix((d, ix, ip), shape=(n, n)).toarray() for ip, ix, d in nep.csr],
                                        nep.terms))
        R.rsrr_sample_gmres(ctx, dn, z, U, zref, tol=args.tol, restart=args.restart, S=S)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            _, dinfo, _ = R.rsrr_sample_gmres(ctx, dn, z, U, zref, tol=args.tol, restart=args.restart, S=S)
        torch.cuda.synchronize()
        dg = (time.perf_counter() - t0) / args.steps
        tmd = ctx.raw_timings()
        dense_op = {"solves_per_s": round(N / dg, 3), "ms_per_step": round(1e3 * dg, 3),
                    "operator_ms": round(tmd[1], 3),
                    "iters_max": max(i["iters"] for i in dinfo),
                    "resid_max": max(i["resid"] for i in dinfo), "converged": all(i["converged"] for i in dinfo)}
        del dn
        torch.cuda.empty_cache()
    if not hasattr(nep, "A") and not sparse:
        # the same solves with the matrix entries generated inside every operator application
        R.rsrr_sample_gmres(ctx, dnep, z, U, zref, tol=args.tol, restart=args.restart, S=S,
                            flags=R.RSRR_GMRES_MATRIX_FREE)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            _, minfo, _ = R.rsrr_sample_gmres(ctx, dnep, z, U, zref, tol=args.tol, restart=args.restart, S=S,
                                              flags=R.RSRR_GMRES_MATRIX_FREE)
        torch.cuda.synchronize()
        dm = (time.perf_counter() - t0) / args.steps
        tmm = ctx.raw_timings()
        mfree = {"solves_per_s": round(N / dm, 3), "ms_per_step": round(1e3 * dm, 3),
                 "operator_ms": round(tmm[1], 3), "setup_ms": round(tmm[0], 3),
                 "resid_max": max(i["resid"] for i in minfo), "converged": all(i["converged"] for i in minfo)}
    gres = {"solves_per_s": round(N / dt, 3), "ms_per_step": round(1e3 * dt, 3),
            "iters_max": max(iters), "iters_mean": round(sum(iters) / len(iters), 2), "cycles": cycles,
            "resid_max": max(i["resid"] for i in info), "converged": all(i["converged"] for i in info),
            "phase_ms": {"setup": round(tm[0], 3), "operator": round(tm[1], 3), "preconditioner": round(tm[2], 3),
                         "krylov_cycles": round(tm[3], 3), "total": round(tm[4], 3)}}
    direct = None
    if not args.no_plain:  # the direct mixed-precision path on the same inputs
        for _ in range(args.warmup):
            R.rsrr_sample(ctx, dnep, z, U, prec=R.RSRR_PREC_C64_IR, S=S)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            _, dinfo, _ = R.rsrr_sample(ctx, dnep, z, U, prec=R.RSRR_PREC_C64_IR, S=S)
        torch.cuda.synchronize()
        dd = (time.perf_counter() - t0) / args.steps
        direct = {"solves_per_s": round(N / dd, 3), "ms_per_step": round(1e3 * dd, 3),
                  "resid_max": max(i["resid"] for i in dinfo)}
    res = {
        "metric": METRIC,
        "value": gres["solves_per_s"],
        "unit": "resolvent solves/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": gres["ms_per_step"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f64 Krylov + operator, c64 LU preconditioner (f32 panels and sums, split-f16 MFMA products)",
        "data": f"synthetic ({getattr(nep, 'name', args.gmres_nep)}, complex Gaussian probes)",
        "config": {"workload": f"GMRES sampling, {args.gmres_nep} n={n}, N={N}, L={L}, "
                               f"{args.nref} reference factorisation(s), restart {args.restart}, tol {args.tol:g}"
                               + (", matrix-free operator" if info[0]["matrix_free"] else ""),
                   "step": "rsrr_sample_gmres over all N points (reference LU, FP64 operator, FGMRES)"},
        "roofline": roof,
        "gmres": gres,
        "gmres_matrix_free": mfree,
        "gmres_dense_operator": dense_op,
        "direct_mixed": direct,
        "gmres_over_direct": round(gres["solves_per_s"] / direct["solves_per_s"], 3) if direct else None,
    }
    print(json.dumps(res), flush=True)


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "the benchmark runs on one GPU only (the sharding across GPUs is a design, not code); run with --gpus 1",
                          "n_gpus_requested": args.gpus}))
        sys.exit(2)
    if args.workload == "serve":
        run_serve(args)
        return
    if args.workload == "batched":
        run_batched(args)
        return
    if args.workload == "adaptive":
        run_adaptive(args)
        return
    if args.workload == "moments":
        run_moments(args)
        return
    if args.workload == "gmres":
        run_gmres(args)
        return
    if args.workload == "real":
        run_real(args)
        return
    import torch
    from paper_1605_07951_amd import rsrr as R

    nep, C, U_host, desc = build_workload(args)
    n, L, N = nep.n, U_host.shape[1], C.N
    dev = torch.device("cuda:0")
    ctx = R.rsrr_create(0)
    dnep = R.DeviceNEP(nep)
    U, _ = R.colmajor(U_host)
    z, _ = R.rsrr_contour(C.gamma, C.a, C.b, N)
    prec = R.RSRR_PREC_C64_IR if args.prec == "mixed" else R.RSRR_PREC_C128
    S = torch.empty((N * L, n), dtype=torch.complex128, device=dev)
    kmax = min(n, N * L)
    radius = max(C.a, C.b)

    def step():
        _, info, _ = R.rsrr_sample(ctx, dnep, z, U, prec=prec, S=S)
        return {"info": info}

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    if args.calib_copy:
        # a plain copy of known size: 1 GiB read, 1 GiB written (reference for the HBM counters)
        src = torch.ones(1 << 28, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    R.rsrr_update_stats(ctx, enable=True, reset=True)
    sample_ms = 0.0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    last = None
    for _ in range(args.steps):
        last = step()
        sample_ms += ctx.timings()["total_ms"]
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    st = R.rsrr_update_stats(ctx, enable=False)
    tm = ctx.timings()

    value = N * args.steps / elapsed
    ms_per_step = 1e3 * elapsed / args.steps
    split = prec == R.RSRR_PREC_C64_IR and n >= SPLIT_MIN_N
    peak = (PEAK_SPLIT_TFLOPS if split else
            PEAK_FP32_MFMA_TFLOPS if prec == R.RSRR_PREC_C64_IR else PEAK_FP64_MFMA_TFLOPS)
    avg_ms = st["ms"] / max(1, st["launches"])
    achieved = (st["flops"] / (st["ms"] * 1e-3) / 1e12) if st["ms"] > 0 else 0.0
    info = last["info"]
    res = {
        "metric": METRIC,
        "value": round(value, 3),
        "unit": "resolvent solves/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c64 LU (f32 panels and sums, split-f16 MFMA updates) + f64 refinement" if prec == R.RSRR_PREC_C64_IR else "c128 (f64 MFMA)",
        "data": "synthetic (seeded Fibonacci-sphere Helmholtz single-layer NEP, complex Gaussian probes)",
        "config": {"workload": desc, "n": n, "N": N, "L": L, "precision": args.prec,
                   "step": "rsrr_sample over all N points (assembly, LU, solves, refinement)"},
        "roofline": {"bound": "mfma", "kernel": "LU trailing update (gemm_split_kernel<float2,true>)" if split else
                     "LU trailing update (cgemm3m_mfma_kernel<4,1,1,2,*,1>)"
                     if prec == R.RSRR_PREC_C64_IR else "LU trailing update (zgemm_mfma_kernel<0,0,128,1>)",
                     "achieved": round(achieved, 3), "peak": round(peak, 1), "unit": "TFLOP/s",
                     "frac": round(achieved / peak, 4),
                     "traffic": (measured_traffic() if (prec == R.RSRR_PREC_C64_IR and args.workload == "helmholtz"
                                                        and n == 4096 and N == 64 and L == 64) else None),
                     "launches": st["launches"], "avg_launch_ms": round(avg_ms, 4),
                     "flops_per_launch": st["flops"] / max(1, st["launches"]),
                     "algorithmic_bytes_per_launch": st["bytes"] / max(1, st["launches"]),
                     **({"cu_masked_part": {
                         "what": "the first columns of each update overlapped with the next panels run on a stream "
                                 "whose CU mask leaves CUs to them: its rate is bounded by that CU share",
                         "cu_share": round(st["masked_cu_share"], 4),
                         "flops_share": round(st["masked_flops"] / st["flops"], 4) if st["flops"] else None,
                         "achieved": round(st["masked_flops"] / (st["masked_ms"] * 1e-3) / 1e12, 3),
                         "frac_of_its_cus": round(st["masked_flops"] / (st["masked_ms"] * 1e-3) / 1e12
                                                  / (peak * st["masked_cu_share"]), 4)}}
                        if st.get("masked_ms", 0) > 0 else {}),
                     **({"form": "split operands: every real FP32 product is three FP16 products with FP32 sums; "
                                 "achieved counts the standard 8 real flops per complex multiply-add, the matrix "
                                 "cores execute 24, and peak is a third of their dense FP16 rate",
                         "mfma_executed_frac": round(achieved / peak, 4),
                         "rocprof_mfma_util": (measured_mfma_util() if (args.workload == "helmholtz" and n == 4096
                                                                        and N == 64 and L == 64) else None)}
                        if split else
                        {"form": "3M: three real MFMA products per complex multiply-add; achieved counts the "
                                 "standard 8 real flops per complex multiply-add, the matrix cores execute 6",
                         "mfma_executed_frac": round(0.75 * achieved / peak, 4)}
                        if prec == R.RSRR_PREC_C64_IR else {})},
        "sample_solves_per_s": round(N * args.steps / (sample_ms * 1e-3), 3) if sample_ms > 0 else None,
        "rhs_columns_per_s": round(L * value, 1),
        "phase_ms_last_step": {k: round(v, 3) for k, v in tm.items()},
        "ir_iters_max": max(i["ir_iters"] for i in info),
        "resid_max": max(i["resid"] for i in info),
        "fallbacks": sum(i["fallback"] for i in info),
    }
    if prec == R.RSRR_PREC_C64_IR and args.workload == "helmholtz":
        res["phase_rooflines"] = phase_rooflines(n, N, L, tm, res["ir_iters_max"])
    if not args.sample_only:
        # the rest of the method on the sampled S: basis, projection, SS-FULL (timed once, reported)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        Q, k, sig = R.rsrr_basis(ctx, S, n, 1e-14, kmax=kmax)
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        AQ, terms = R.rsrr_project(ctx, dnep, Q, k, C.gamma, radius)
        torch.cuda.synchronize()
        t3 = time.perf_counter()
        sol = R.rsrr_solve(ctx, dnep, Q, k, AQ, terms, C.gamma, C.a, C.b, NQ=args.nq, KQ=2)
        torch.cuda.synchronize()
        t4 = time.perf_counter()
        d = sol["lam"] - complex(C.gamma)
        lv = (d.real / C.a) ** 2 + (d.imag / C.b) ** 2   # elliptic level: < 1 inside the contour
        ins = lv < 1
        res["rest_of_method"] = {"basis_ms": round(1e3 * (t2 - t1), 1), "project_ms": round(1e3 * (t3 - t2), 1),
                                 "solve_ms": round(1e3 * (t4 - t3), 1), "k": k, "terms": len(terms),
                                 "nbar": sol["nbar"], "gmax": sol["gmax"], "eigs_inside": int(ins.sum()),
                                 "eig_resid_max_inside": float(sol["resid"][ins].max()) if ins.any() else None,
                                 "lambda_inside": [[float(l.real), float(l.imag)] for l in sol["lam"][ins]]}
        # latency of the whole method for one NEP (sampling, basis, projection, SS-FULL), repeated
        lat = []
        for _ in range(args.latency_runs):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            R.rsrr_sample(ctx, dnep, z, U, prec=prec, S=S)
            Q, k, _ = R.rsrr_basis(ctx, S, n, 1e-14, kmax=kmax)
            AQ, terms = R.rsrr_project(ctx, dnep, Q, k, C.gamma, radius)
            R.rsrr_solve(ctx, dnep, Q, k, AQ, terms, C.gamma, C.a, C.b, NQ=args.nq, KQ=2)
            torch.cuda.synchronize()
            lat.append(time.perf_counter() - t0)
        if lat:
            res["nep_latency_s"] = {"p50": round(_pct(lat, 50), 4), "p99": round(_pct(lat, 99), 4),
                                    "mean": round(sum(lat) / len(lat), 4), "runs": len(lat),
                                    "what": "one NEP alone, whole method: rsrr_sample + rsrr_basis + rsrr_project"
                                            " + rsrr_solve (eigenpairs and residuals on the host)"}

    if not args.no_plain and prec == R.RSRR_PREC_C64_IR:
        # plain FP64 path on the same inputs for the mixed/plain speedup, with the roofline of its
        # trailing update (FP64 MFMA, 4M form: 8 m^2 k flops per complex update, all on the matrix cores)
        R.rsrr_sample(ctx, dnep, z, U, prec=R.RSRR_PREC_C128, S=S)
        torch.cuda.synchronize()
        R.rsrr_update_stats(ctx, enable=True, reset=True)
        t1 = time.perf_counter()
        R.rsrr_sample(ctx, dnep, z, U, prec=R.RSRR_PREC_C128, S=S)
        torch.cuda.synchronize()
        dtp = time.perf_counter() - t1
        pst = R.rsrr_update_stats(ctx, enable=False)
        ptm = ctx.timings()
        res["plain_c128_sample_solves_per_s"] = round(N / dtp, 3)
        if res["sample_solves_per_s"]:
            res["mixed_over_plain_speedup"] = round(res["sample_solves_per_s"] / (N / dtp), 3)
        if pst["ms"] > 0:
            pach = pst["flops"] / (pst["ms"] * 1e-3) / 1e12
            lu_all = N * (8.0 / 3.0) * float(n) ** 3
            res["plain_c128_roofline"] = {
                "bound": "mfma", "kernel": "LU trailing update, complex FP64 (zgemm_mfma_kernel<0,0,128,1>)",
                "achieved": round(pach, 3), "peak": PEAK_FP64_MFMA_TFLOPS, "unit": "TFLOP/s",
                "frac": round(pach / PEAK_FP64_MFMA_TFLOPS, 4), "launches": pst["launches"],
                "avg_launch_ms": round(pst["ms"] / max(1, pst["launches"]), 4),
                "flops_per_launch": pst["flops"] / max(1, pst["launches"]),
                "lu_phase_ms": round(ptm["lu_ms"], 3),
                "lu_phase_TFLOP_s": round(lu_all / (ptm["lu_ms"] * 1e-3) / 1e12, 3) if ptm["lu_ms"] > 0 else None,
                "phase_ms": {k: round(v, 3) for k, v in ptm.items()}}

    if args.serve_leg > 0 and args.workload == "helmholtz" and prec == R.RSRR_PREC_C64_IR:
        # p50/p99 under load: the first requests of the seeded serving stream at the stated 20/s
        # (over capacity: backlog) and at a sustainable rate
        del S
        ctx.close()
        torch.cuda.empty_cache()
        items = serving_items(args.serve_leg, args.rate)
        fast, _ = serve_stream(items, "20/s", R.RSRR_PREC_C64_IR, 0, args.slots, args.arena_gb, args.batch_gb,
                               args.solvers)
        slow, _ = serve_stream(items, "sustainable", R.RSRR_PREC_C64_IR, 0, args.slots, args.arena_gb,
                               args.batch_gb, args.solvers, rate_scale=args.serve_slow_rate / args.rate)
        res["serving"] = {"what": f"first {len(items)} requests of the seeded serving stream (50/50 delay n "
                                  f"512/1024/2048 N=48 L=32 / Helmholtz n 2048/4096/8192 N=64 L=64), whole "
                                  f"method per request, latency = submission to eigenpairs on the host",
                          "rate_20_per_s": fast, f"rate_{args.serve_slow_rate:g}_per_s": slow}
        del items

    if not args.no_cpu:
        npts = args.cpu_points or (4 if n >= 2048 else min(N, 16))
        res["cpu_baseline"] = cpu_baseline(nep, C, U_host, npts)
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
