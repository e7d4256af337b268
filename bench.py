#!/usr/bin/env python3
"""Benchmark: ADMM-BB iterations/s on the 13-scenario head-and-neck-shaped workload.

One step = one full ADMM-BB iteration of the hot path for all 13 scenarios:
gradient/objective pass at z (residual of the x-update system), up to cg_max
warm-started CG steps per scenario (each a fused A_s^T W A_s pass), z-update,
residual norms, Barzilai-Borwein step and dual update.  Inputs are resident in
HBM before the timed region starts (setup is timed separately).

Prints one JSON line.  Also reports time-to-1e-5 relative objective gap against
the oracle's exact minimum (stored reference, checked by content digest), the
fused-pass roofline, and the FP64 CPU oracle timed on this host.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--precision fp32|bf16|fp16]
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "time-to-1e-5 obj (s) & ADMM iters/s, 13 scen.; SpMV HBM GB/s vs ~8 TB/s"
HBM_PEAK_GBS = 8000.0
# HBM bytes per launch of the dense x-update kernel (k_dense_x: the packed
# tiles of every inverse, beside the previous iteration's stopping test) on
# this workload, from rocprofv3 FETCH_SIZE (x 2.0) and WRITE_SIZE (x 1.0) runs
# (profiles/k_dense_x_hn13_fp32.md); valid only while the text of the tile
# function and of the kernel is the one they were taken with (the two 16-digit
# hashes of kernel_source_hash)
XSYM_TRAFFIC = {"source_hashes": "4a8933afcacabecb4aa3b36fee9001bb", "fetch_bytes": 119699.5 * 1024 * 2.0,
                "write_bytes": 14358.7 * 1024 * 1.0}


def kernel_source_hash(path: str, signature: str) -> str:
    """sha256 (16 hex digits) of one kernel's text: from its signature to the closing brace."""
    src = open(path).read()
    a = src.find(signature)
    if a < 0:
        return ""
    b = src.find("\n}\n", a) + 3
    return hashlib.sha256(src[a:b].encode()).hexdigest()[:16]


def pass_bytes(P, precision: str) -> np.ndarray:
    """Algorithmic bytes of one fused CG pass over each scenario's A_s:
    per nonzero the value (4 B fp32, 2 B bf16/fp16) and a 2 B column index;
    per nonempty row a 4 B row offset and a 4 B weight (plus a 4 B scale for
    bf16/fp16); the n-vector read once and its column sums written once."""
    vb = 4 if precision == "fp32" else 2
    rowb = 8 if precision == "fp32" else 12
    out = []
    for a in P.A:
        rows = int(np.count_nonzero(np.diff(a.row_ptr)))
        out.append(a.nnz * (vb + 2) + rows * rowb + 4 + 8 * P.n)
    return np.asarray(out, dtype=np.float64)


def spmv_bytes(P) -> dict:
    """Algorithmic bytes of one sparse pass over all scenarios (fp32 values, u16
    columns): per nonzero 6 B; per nonempty row the chunk offset plus two 4 B
    row values (weight and prescription for the forward pass, original index and
    the gathered t_i for the transpose); the n-vector in or out."""
    out = {}
    tot = 0.0
    for a in P.A:
        rows = int(np.count_nonzero(np.diff(a.row_ptr)))
        tot += a.nnz * 6 + rows * 12 + 4 * P.n
    out["forward"] = tot
    out["transpose"] = tot
    out["normal"] = float(pass_bytes(P, "fp32").sum())
    return out


def host_triad() -> dict:
    """The host's memory roofline: a STREAM-style triad a = b + s c over three
    1 GiB float64 arrays with PyTorch's CPU thread pool, best of three; 24
    bytes per element (two reads, one write)."""
    import torch
    n = 1 << 27
    b = torch.full((n,), 1.0, dtype=torch.float64)
    c = torch.full((n,), 2.0, dtype=torch.float64)
    a = torch.empty_like(b)
    best = float("inf")
    for _ in range(3):
        t0 = time.perf_counter()
        torch.add(b, c, alpha=3.0, out=a)
        best = min(best, time.perf_counter() - t0)
    return {"GB/s": 24.0 * n / best / 1e9, "threads": torch.get_num_threads()}


def cpu_baseline(P, fstar, budget_s: float = 90.0, progress: bool = False) -> dict:
    """Time the FP64 oracle's ADMM-BB (the paper's algorithm: cached Cholesky
    x-updates, Appendix A) on the whole workload, all 13 scenarios, on this
    host: the set-up (dense Gram matrix and Cholesky factor per scenario), then
    iterations from zero until (f - f*)/f* <= 1e-5 against the stored oracle
    minimum, stopped by the oracle's own per-iteration callback.  The oracle is
    used as it stands: its scenario loop is serial, so the cores it actually
    keeps busy are measured (process CPU time over wall time) next to the BLAS
    thread pool it may use.  A second, short run limited to one BLAS thread
    gives the single-thread iteration rate."""
    from oracle import admm as oadmm, wls as owls
    try:
        from threadpoolctl import threadpool_info, threadpool_limits
        blas_threads = max([t.get("num_threads", 1) for t in threadpool_info()] + [1])
    except Exception:  # pragma: no cover
        threadpool_limits = None
        blas_threads = os.cpu_count() or 1

    class _Done(Exception):
        pass

    W = owls.from_problem(P)
    c0, t0 = time.process_time(), time.perf_counter()
    S = oadmm.AdmmSetup(W, owls.default_rho(W))
    t_setup = time.perf_counter() - t0
    cpu_setup = time.process_time() - c0
    stamps = []
    t_start = time.perf_counter()

    def cb(k, z, f):
        stamps.append((k + 1, time.perf_counter(), f))
        if progress:
            print(f"[cpu] iteration {k + 1}: {time.perf_counter() - t_start:.1f} s", file=sys.stderr, flush=True)
        if fstar is not None and (f - fstar) / fstar <= 1e-5:
            raise _Done
        if time.perf_counter() - t_start > budget_s:
            raise _Done

    c1 = time.process_time()
    try:
        oadmm.admm_bb(W, setup=S, max_iter=5000, record=False, callback=cb)
    except _Done:
        pass
    solve_s = time.perf_counter() - t_start
    cpu_solve = time.process_time() - c1
    iters, _, f_last = stamps[-1]
    reached = fstar is not None and (f_last - fstar) / fstar <= 1e-5
    # single BLAS thread: a few iterations, rate from the callback stamps
    one = []
    if threadpool_limits is not None:
        with threadpool_limits(limits=1):
            oadmm.admm_bb(W, setup=S, max_iter=4, obj_rel_tol=0.0, eps_abs=0.0, eps_rel=0.0, record=False,
                          callback=lambda k, z, f: one.append(time.perf_counter()))
    rate1 = (len(one) - 1) / (one[-1] - one[0]) if len(one) > 1 else None
    busy = (cpu_setup + cpu_solve) / (t_setup + solve_s)
    return {"value": iters / solve_s, "unit": "ADMM iter/s", "cores": int(math.ceil(busy - 1e-9)), "kind": "oracle",
            "sample": f"FP64 oracle ADMM-BB (cached Cholesky x-updates) on the whole workload, all "
                      f"{P.num_scen} scenarios: set-up {t_setup:.1f} s, then {iters} iterations from zero in "
                      f"{solve_s:.1f} s" + (" to the 1e-5 objective gap" if reached else
                                             " (time budget; the 1e-5 gap was not reached)"),
            "setup_s": t_setup, "solve_s": solve_s, "iters": int(iters),
            "time_to_1e-5_s": (t_setup + solve_s) if reached else None,
            "time_to_1e-5_solve_only_s": solve_s if reached else None,
            "reached_1e-5": bool(reached), "blas_threads": int(blas_threads),
            "cpu_busy_cores": busy, "iter_per_s_1_thread": rate1, "host_triad": host_triad()}


def cpu_scaling(args):
    """The oracle's side of the scenario-count study (Sec. 3.3): cpu_baseline on
    the workload restricted to its first N scenarios, against the stored oracle
    minimum of each restriction, and on the two smallest patients of the batch
    recipe with their 64-scenario lattice."""
    import synth
    from paper_2304_14568_amd.refdata import load as load_ref
    P_all = synth.hn_full(args.seed)
    rows = []
    for N in [int(v) for v in args.cpu_scaling.split(",")]:
        P = P_all.subset(list(range(N)))
        name = f"hn_full_s{args.seed}" if N == P_all.num_scen else f"hn_full_s{args.seed}_n{N}"
        rec, _ = load_ref(name)
        fstar = rec["f_star"] if (rec is not None and rec["digest"] == P.digest()) else None
        r = cpu_baseline(P, fstar, budget_s=300.0, progress=True)
        r.update(N=N, workload=name)
        rows.append(r)
        print(f"[cpu-scaling] N={N}: set-up {r['setup_s']:.1f}s, {r['iters']} it in {r['solve_s']:.1f}s",
              file=sys.stderr, flush=True)
    for k in (2, 1):
        P = synth.batch_patient(k, num=8, scen=64, seed=10)
        rec, _ = load_ref(f"batch_s10_p{k}")
        if rec is None or rec["digest"] != P.digest():
            continue
        print(f"[cpu-scaling] batch patient {k}: oracle set-up of {P.num_scen} scenarios", file=sys.stderr,
              flush=True)
        r = cpu_baseline(P, rec["f_star"], budget_s=600.0, progress=True)
        r.update(N=P.num_scen, workload=f"batch_s10_p{k}", m=P.m, n=P.n)
        rows.append(r)
        print(f"[cpu-scaling] batch patient {k} (N={P.num_scen}): set-up {r['setup_s']:.1f}s, {r['iters']} it in "
              f"{r['solve_s']:.1f}s", file=sys.stderr, flush=True)
        break
    print(json.dumps({"kind": "oracle scenario-count scaling", "rows": rows}), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=500)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--precision", default="fp32", choices=["fp32", "bf16", "fp16"])
    ap.add_argument("--format", default="auto", choices=["auto", "csr", "sell"],
                    help="layout of A_s for the sparse passes (auto: the set-up autotuner picks)")
    ap.add_argument("--cg-max", type=int, default=8)
    ap.add_argument("--dense-launches", type=int, default=3, choices=[3, 4],
                    help="dense x-update: three launches per iteration (default) or four, each iteration complete at its end")
    ap.add_argument("--xupdate", default="auto", choices=["auto", "cg", "dense"],
                    help="x-update: warm-started CG on the sparse A_s, or the cached dense inverse")
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--no-ttt", action="store_true", help="skip the time-to-tolerance measurement")
    ap.add_argument("--calib-copy-mib", type=int, default=0,
                    help="first copy this many MiB device-to-device (a reference kernel for HBM byte counters)")
    ap.add_argument("--graph", action="store_true",
                    help="with --xupdate cg, replay each iteration from a captured HIP graph in the throughput "
                         "region (the instrumented region and the dense iterations always launch directly)")
    ap.add_argument("--cpu-scaling", default="",
                    help="only time the FP64 oracle (set-up and iterations to the 1e-5 gap) on the first N "
                         "scenarios of the workload for each N of this comma-separated list, and on the "
                         "64-scenario lattice patients with stored minima; print one JSON line")
    args = ap.parse_args()
    if args.cpu_scaling:
        return cpu_scaling(args)
    if args.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU; multi-GPU scenario sharding is a design "
                                   "note only (one all-reduce of an n-vector per iteration)", "n_gpus": args.gpus}))
        sys.exit(2)

    import torch
    import synth
    import paper_2304_14568_amd as A
    from paper_2304_14568_amd.refdata import load as load_ref

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    stream = torch.cuda.Stream(device=dev)

    if args.calib_copy_mib > 0:
        src = torch.ones(args.calib_copy_mib * 1024 * 1024 // 4, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    t0 = time.perf_counter()
    P = synth.hn_full(args.seed)
    t_gen = time.perf_counter() - t0
    digest = P.digest()
    ref, xstar = load_ref(f"hn_full_s{args.seed}")
    fstar = ref["f_star"] if (ref is not None and ref["digest"] == digest) else None

    # the process's GPU runtime start-up (paid once per process, by whatever
    # touches the device first) stays outside the solver's set-up time
    torch.zeros(1, device=dev).add_(1.0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    S = A.Solver(P, precision=args.precision, cg_max=args.cg_max, max_iter=2000, stream=stream,
                 use_graph=1 if args.graph else 0, xupdate=args.xupdate, format=args.format,
                 dense_launches=args.dense_launches)
    torch.cuda.synchronize()
    t_setup = time.perf_counter() - t0
    xmode, factor_ms = S.xupdate()

    # warm-up: graph capture, caches, clocks
    S.iterate(max(1, args.warmup))
    # throughput region: K iterations from zero initialisation, no instrumentation
    S.reset()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    info = S.iterate(args.steps)
    torch.cuda.synchronize()
    t_run = time.perf_counter() - t0
    iters_per_s = args.steps / t_run
    # instrumented region: the same K iterations with HIP events around every
    # fused CG pass launch (on the library's stream)
    S.reset()
    S.enable_timing(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    S.iterate(args.steps)
    torch.cuda.synchronize()
    t_inst = time.perf_counter() - t0
    tm = S.timing()
    counts = S.cg_counts()
    S.enable_timing(False)

    if xmode == "dense":
        # x-update roofline: every launch reads each scenario's packed fp32
        # inverse once (upper 64 x 64 tiles of M_s, 16 KiB each) and its fp64
        # right-hand side; in the three-launch order the same launch (k_dense_x)
        # runs the previous iteration's stopping test in its first workgroup
        nb = (P.n + 63) // 64
        tiles = nb * (nb + 1) // 2
        bytes_per_launch = float(P.num_scen * (tiles * 64 * 64 * 4 + 8 * P.n))
        launches = tm["pass_launches"]
        achieved = bytes_per_launch / (tm["pass_ms"] * 1e-3) / 1e9 if tm["pass_ms"] > 0 else 0.0
        traffic = None
        src = os.path.join(ROOT, "paper_2304_14568_amd", "csrc", "factor.hip")
        if (args.seed == 0 and args.dense_launches == 3 and os.path.exists(src) and
                XSYM_TRAFFIC["source_hashes"] is not None and
                kernel_source_hash(src, "__device__ __forceinline__ void xsym_tile(") +
                kernel_source_hash(src, "__global__ __launch_bounds__(256) void k_dense_x(") ==
                XSYM_TRAFFIC["source_hashes"]):
            traffic = XSYM_TRAFFIC["fetch_bytes"] + XSYM_TRAFFIC["write_bytes"]
        kname = ("k_dense_x (x_s = M_s c_s over the packed upper tiles of the cached fp32 inverses, beside the "
                 "previous iteration's stopping test)" if args.dense_launches == 3 else
                 "k_xsym (x_s = M_s c_s over the packed upper tiles of the cached fp32 inverses)")
        roof = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": achieved / HBM_PEAK_GBS, "traffic": traffic, "kernel": kname,
                "avg_launch_ms": tm["pass_ms"], "launches": launches, "bytes_per_launch": bytes_per_launch}
    else:
        # fused CG pass roofline: algorithmic bytes of the scenario passes actually
        # performed / summed duration of all CG pass launches in the timed region
        pb = pass_bytes(P, args.precision)
        total_bytes = float(np.dot(counts, pb))
        pass_time_s = tm["pass_ms"] * tm["pass_launches"] * 1e-3
        achieved = total_bytes / pass_time_s / 1e9 if pass_time_s > 0 else 0.0
        launches = tm["pass_launches"]
        roof = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": achieved / HBM_PEAK_GBS, "traffic": None,
                "kernel": "k_pass (fused CG pass A_s^T diag(c_s w) A_s v)",
                "avg_launch_ms": tm["pass_ms"], "launches": launches,
                "bytes_per_full_pass": float(pb.sum()), "scenario_passes": int(counts.sum())}

    result = {
        "metric": METRIC,
        "value": iters_per_s,
        "unit": "ADMM iter/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1e3 * t_run / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32" if args.precision == "fp32" else f"{args.precision}+f32",
        "data": "synthetic",
        "config": {"workload": f"head-and-neck-shaped phantom seed {args.seed}: 120x120x80 grid at 2.5 mm, "
                               f"{P.m} body voxels, {P.n} spots (3 beams x 15 layers), 13 scenarios",
                   "m": P.m, "n": P.n, "scenarios": P.num_scen, "nnz": P.nnz, "precision": args.precision,
                   "cg_max": args.cg_max, "xupdate": xmode, "dense_launches": args.dense_launches,
                   "parallelism": "single GPU, all scenarios per launch"},
        "roofline": roof,
        "instrumented_ms_per_step": 1e3 * t_inst / args.steps,
        "graph": bool(args.graph),
        "tuning": S.tuning(),
        "setup_s": t_setup,
        "dense_factor_ms": factor_ms if xmode == "dense" else None,
        "generate_s": t_gen,
        "obj_after_steps": info[0]["obj"],
    }

    # what the memory system delivers for one streaming read at the sizes that
    # matter here: the dense iteration's working set (inverses + sum of Gram
    # matrices + partials, re-read every iteration) and a stream well beyond the
    # 256 MB last-level cache
    if xmode == "dense":
        # packed inverses + packed fp64 sum of the Gram matrices + fp64 tile partials
        ws_bytes = int(bytes_per_launch + tiles * 64 * 64 * 8 + P.num_scen * tiles * 128 * 8)
    else:
        ws_bytes = int(pass_bytes(P, args.precision).sum())
    probe = {}
    for label, nb in (("working_set", ws_bytes), ("1GiB", 1 << 30)):
        if nb >= (1 << 20):
            probe[label] = {"bytes": nb, "GB/s": A.stream_probe(nb, reps=10)}
    result["stream_probe"] = probe
    if "working_set" in probe:
        roof["frac_of_stream_probe"] = roof["achieved"] / probe["working_set"]["GB/s"]

    # the sparse products on their own (dense and CG x-updates alike use them for
    # the objective, gradients, features and the CG operator)
    sb = spmv_bytes(P)
    spmv = {}
    for kind in ("forward", "transpose", "normal"):
        ms = S.time_pass(kind, reps=20)
        gbs = sb[kind] / (ms * 1e-3) / 1e9
        spmv[kind] = {"ms": ms, "bytes": sb[kind], "GB/s": gbs, "frac": gbs / HBM_PEAK_GBS}
    result["spmv"] = spmv

    if not args.no_ttt:
        # time to reach (f - f*) / f* <= 1e-5 from zero initialisation
        S.reset()
        zs, sinfo, st = S.solve()
        trace = S.trace()
        result["solve_paper_stop"] = {"iters": sinfo[0]["iter"], "status": int(st), "obj": sinfo[0]["obj"],
                                      "r_prim": sinfo[0]["r_prim"], "eps_prim": sinfo[0]["eps_prim"],
                                      "r_dual": sinfo[0]["r_dual"], "eps_dual": sinfo[0]["eps_dual"]}
        if fstar is not None:
            k_hit = next((t["iter"] for t in trace if (t["obj"] - fstar) / fstar <= 1e-5), None)
            result["f_star"] = fstar
            result["final_rel_gap"] = (sinfo[0]["obj"] - fstar) / fstar
            result["z_rel_err_l2"] = float(np.linalg.norm(zs[0] - xstar) / np.linalg.norm(xstar))
            if k_hit is not None:
                S.reset()
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                S.iterate(k_hit)
                torch.cuda.synchronize()
                result["time_to_1e-5_s"] = time.perf_counter() - t0
                result["iters_to_1e-5"] = k_hit
                # the same, counted from the start of the set-up (validation, packing,
                # upload, cached inverses)
                result["time_to_1e-5_from_setup_s"] = t_setup + result["time_to_1e-5_s"]
            else:
                result["time_to_1e-5_s"] = None
        else:
            result["f_star"] = None
            result["note"] = "stored oracle reference missing or digest mismatch: no time-to-tolerance"

    if not args.no_cpu:
        result["cpu_baseline"] = cpu_baseline(P, fstar)
    S.close()
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
