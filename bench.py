"""Benchmark: graph-form ADMM on one MI355X.

Default line (``python bench.py``): one step = one whole solve of the Lasso
20000 x 2000 workload with A already resident in HBM: pogs_init (layout,
Sinkhorn-Knopp equilibration, Frobenius normalisation, MFMA Gram, float64
Cholesky and inverse) + pogs_solve (the ADMM iterations until the stopping
test passes at eps_abs = 1e-4, eps_rel = 1e-3) + pogs_free.  value = solves/s
(converged solves only), with ADMM iter/s, p50/p99 step latency, the roofline
of the dominant per-iteration kernel (HIP events on the library's stream),
the FP64 CPU oracle's rate on the host cores and the objective's error
against that oracle.  Beside it, each against its plain one-problem path on
the same GPU and with its objective error against the oracle:
  dose     the dose-shaped 100000 x 1000 problem (whole solves, roofline);
  batched  512 uneven Lasso/logistic problems in one batch call;
  path     a 64-point lambda path on one 8000 x 1000 matrix;
  serving  mixed requests through the serving engine (closed loop, then
           Poisson arrivals at 80 % of it: p50/p99 latency).

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-blocks]
                    [--workload lasso|nnls|dose|lasso-cgls|batch|path|serve|sparse]
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0  # MI355X HBM3E, GB/s

WORKLOADS = {  # name: (generator, description, projection)
    "lasso": ("lasso_20000x2000", "Lasso 20000x2000 float32, lambda = 0.1 ||A^T b||_inf", "direct"),
    "nnls": ("nnls_20000x2000", "NNLS 20000x2000 float32 (same A, b as the Lasso)", "direct"),
    "dose": ("dose_100000x1000", "dose-shaped 100000x1000 float32, 30% |N(0,1)| dense, asym. L1, x >= 0", "direct"),
    "lasso-cgls": ("lasso_20000x2000", "Lasso 20000x2000 float32, CGLS projection (no Gram, no factor)", "cgls"),
}

# HBM traffic of the dominant kernel, from rocprofv3 FETCH_SIZE / WRITE_SIZE
# runs summarised in profiles/ (record lines "traffic workload=... kernel=...
# sources=<digest> bytes=<per launch>").  A record counts only while the
# sources that define the kernel, its epilogue and its launch shape are the
# ones it was taken on.
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic_lasso_20000x2000.md")
KERNEL_SOURCES = [os.path.join("paper_1503_08366_amd", "csrc", f)
                  for f in ("common.hpp", "gemv.hpp", "gemv_launch.hpp", "iter.hpp", "iter.hip", "internal.hpp",
                            "ctx.hpp")]


def kernel_sources_digest() -> str:
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def recorded_traffic(workload: str, kernel: str):
    try:
        with open(TRAFFIC_FILE) as fh:
            text = fh.read()
    except OSError:
        return None
    digest = kernel_sources_digest()
    for rec in re.finditer(r"traffic workload=(\S+) kernel=(\S+) sources=([0-9a-f]+) bytes=(\d+)", text):
        if rec.group(1) == workload and rec.group(2) == kernel and rec.group(3) == digest:
            return int(rec.group(4))
    return None


def _cpu_threads() -> int:
    try:
        from threadpoolctl import threadpool_info
        info = threadpool_info()
        n = max((d.get("num_threads", 0) for d in info if d.get("user_api") == "blas"), default=0)
        if n:
            return int(n)
    except Exception:
        pass
    return os.cpu_count() or 1


def cpu_baseline(prob, budget_s: float = 30.0, projection: str = "direct"):
    """The FP64 oracle (NumPy/SciPy) on the host: whole solves of the same
    problem, repeated while under the time budget (at least one)."""
    from oracle import pogs_oracle as O
    prm = O.Params(eps_abs=prob.eps_abs, eps_rel=prob.eps_rel, max_iter=prob.max_iter,
                   eps_cmp=float(np.finfo(np.float32).eps), projection=projection)
    A64 = prob.A.astype(np.float64)
    done = 0
    t0 = time.perf_counter()
    iters = 0
    while True:
        r = O.solve(A64, prob.f, prob.g, prm)
        done += 1
        iters += r.iters
        if time.perf_counter() - t0 > budget_s / 2 or done >= 3:
            break
    dt = time.perf_counter() - t0
    return {"value": done / dt, "unit": "solves/s", "cores": _cpu_threads(), "kind": "oracle",
            "sample": f"{done} whole solve(s) of the same workload in FP64 ({iters} ADMM iterations, "
                      f"{dt:.1f} s)", "iter_per_s": iters / dt, "optval": float(r.optval),
            "converged": bool(r.converged)}


def rel_err(got: float, ref: float) -> float:
    """Objective error against the oracle: |p - p_oracle| / max(|p_oracle|, 1)."""
    return abs(got - ref) / max(abs(ref), 1.0)


GOLDEN_DIR = os.path.join(ROOT, "tests", "golden")


def stored_oracle(name: str, probs):
    """Oracle objectives stored by tests/golden/make_golden.py (FP64 oracle
    only), or None unless every record was computed on exactly these inputs."""
    from paper_1503_08366_amd import workloads as W
    try:
        with open(os.path.join(GOLDEN_DIR, name)) as fh:
            recs = json.load(fh)["results"]
    except (OSError, ValueError, KeyError):
        return None
    if len(recs) != len(probs) or any(r["fingerprint"] != W.fingerprint(p) for r, p in zip(recs, probs)):
        return None
    return recs


def err_summary(res, recs):
    if recs is None:
        return None
    e = np.array([rel_err(r.optval, g["optval"]) for r, g in zip(res, recs)])
    return {"max": float(e.max()), "median": float(np.median(e)), "count": int(e.size),
            "oracle": "stored FP64-oracle objectives (tests/golden/)"}


def bench_batch(args):
    """512 uneven Lasso/logistic problems: one batched call vs one problem per launch sequence."""
    from paper_1503_08366_amd import pogs as P
    from paper_1503_08366_amd import workloads as W
    block = batch_block(P, W.batch_mix(count=args.count), args.plain_count)
    return {"metric": "solves/s at rel tol 1e-3, batched (grouped launches per phase) vs plain",
            "value": block["solves_per_s"], "unit": "solves/s", "n_gpus": 1, "higher_is_better": True,
            "config": {"workload": block["workload"]}, **block}


def batch_block(P, probs, plain_count, reps=2):
    """The batch call over all problems (grouped launches: one launch per phase
    for every problem) against the plain path, one pogs_init + pogs_solve per
    problem; both from host inputs, the plain leg without the load-policy
    tuner (the batched leg has none)."""
    recs = stored_oracle("batch_mix_512.json", probs) if len(probs) == 512 else None
    P.pogs_solve_batch(probs)  # warm at full size (device memory pool, pinned ring)
    tb = []
    for _ in range(reps):
        t = time.perf_counter()
        res = P.pogs_solve_batch(probs)
        tb.append(time.perf_counter() - t)
    tb = float(np.mean(tb))
    conv = sum(r.converged for r in res)
    nplain = min(len(probs), plain_count)
    prm = P.default_params(autotune=0)
    t = time.perf_counter()
    plain_conv = 0
    for p in probs[:nplain]:
        with P.Context(p.A, prm) as ctx:
            plain_conv += ctx.solve(p.f, p.g, prm).converged
    tp = time.perf_counter() - t
    return {"workload": f"{len(probs)} problems, even Lasso / odd logistic, m~U[64,4096], n~U[32,1024], "
                        "float32, host inputs (PCIe copy inside the timed region for both legs)",
            "solves_per_s": conv / tb, "seconds": tb, "converged": f"{conv}/{len(res)}",
            "iters_mean": float(np.mean([r.iters for r in res])),
            "plain": {"solves_per_s": plain_conv / tp, "seconds": tp, "problems": nplain,
                      "converged": f"{plain_conv}/{nplain}", "autotune": 0},
            "speedup": (conv / tb) / max(plain_conv / tp, 1e-30),
            "oracle_rel_err": err_summary(res, recs)}


def bench_path(args):
    """64-point lambda path on one 8000x1000 A: stacked right-hand sides on MFMA vs one solve per lambda."""
    from paper_1503_08366_amd import pogs as P
    from paper_1503_08366_amd import workloads as W
    block = path_block(P, W.lambda_path(R=args.R))
    return {"metric": "solves/s at rel tol 1e-3, lambda path (stacked RHS, MFMA) vs plain",
            "value": block["solves_per_s"], "unit": "solves/s", "n_gpus": 1, "higher_is_better": True,
            "config": {"workload": block["workload"]}, **block}


def path_block(P, probs):
    """All lambdas of one path in one call (shared A, K^-1; the passes are
    MFMA products over the stacked right-hand sides) against one solve per
    lambda on the same context; shared setup excluded from both legs."""
    recs = stored_oracle("lambda_path_8000x1000.json", probs)
    with P.Context(probs[0].A) as ctx:
        # warm both legs at full size (device memory pool, captured graphs,
        # the host pool that packs the functions: its second call is still
        # slower), then the median of three path calls
        for _ in range(2):
            ctx.solve_path([p.f for p in probs], [p.g for p in probs])
        ctx.solve(probs[0].f, probs[0].g)
        tp = []
        for _ in range(3):
            t = time.perf_counter()
            res = ctx.solve_path([p.f for p in probs], [p.g for p in probs])
            tp.append(time.perf_counter() - t)
        tpath = sorted(tp)[1]
        t = time.perf_counter()
        alone = [ctx.solve(p.f, p.g) for p in probs]
        tplain = time.perf_counter() - t
        setup_ms = alone[0].ms_setup
    conv = sum(r.converged for r in res)
    return {"workload": f"{len(probs)} Lasso lambdas log-spaced over [1e-3, 1] lam_max, A 8000x1000 float32, "
                        "shared setup excluded from both legs", "setup_ms": setup_ms,
            "solves_per_s": conv / tpath, "seconds": tpath, "seconds_samples": tp, "converged": f"{conv}/{len(res)}",
            "iters_max": max(r.iters for r in res),
            "plain": {"seconds": tplain, "solves_per_s": sum(r.converged for r in alone) / tplain,
                      "iters_sum": sum(r.iters for r in alone)},
            "speedup": tplain / tpath, "oracle_rel_err": err_summary(res, recs)}


def bench_sparse(args):
    """Sparse Lasso 2,000,000 x 200,000 with 16 entries per row (32M entries),
    CGLS projection.  The context (host validation, transpose, upload,
    equilibration) is created once and its time reported; the timed steps are
    whole solves on it."""
    from paper_1503_08366_amd import pogs as P
    from paper_1503_08366_amd import workloads as W
    prob = W.sparse_problem("lasso", 2_000_000, 200_000, 16, seed=5)
    m, n, nnz = prob.m, prob.n, prob.A.nnz
    prm = P.default_params(eps_abs=prob.eps_abs, eps_rel=prob.eps_rel, max_iter=prob.max_iter)
    t = time.perf_counter()
    ctx = P.SparseContext(prob.A, prm)
    setup_s = time.perf_counter() - t
    try:
        for _ in range(args.warmup):
            ctx.solve(prob.f, prob.g, prm, device_out=True)
        lat, res = [], []
        t0 = time.perf_counter()
        for _ in range(args.steps):
            t = time.perf_counter()
            res.append(ctx.solve(prob.f, prob.g, prm, device_out=True))
            lat.append(time.perf_counter() - t)
        total = time.perf_counter() - t0
        prof = ctx.profile_iteration(args.profile_reps)
    finally:
        ctx.free()
    iters = sum(r.iters for r in res)
    # one CG step: the entries of A^ and A^T (value and 16-bit index in its
    # segment), and the vectors the two passes read and write
    alg_bytes = 2.0 * 6 * nnz + 4.0 * (5 * m + 8 * n)
    achieved = alg_bytes / (prof["cg_step"] * 1e-3) / 1e9
    return {"metric": "solves/s at rel tol 1e-3 on a sparse A (CGLS projection, context reused)",
            "value": sum(r.converged for r in res) / total, "unit": "solves/s", "n_gpus": 1,
            "steps": args.steps, "warmup": args.warmup, "ms_per_step": 1e3 * total / args.steps,
            "higher_is_better": True, "dtype": "f32 values, int32 indices, f64 accumulation",
            "data": "synthetic (seeded, 16 uniform columns per row)",
            "config": {"workload": f"sparse Lasso {m}x{n}, {nnz} entries", "nnz": nnz,
                       "setup_s": setup_s, "input": "host CSR"},
            "iters_per_solve": iters / len(res), "cg_steps_per_iteration": sum(r.cg_steps for r in res) / max(iters, 1),
            "converged": f"{sum(r.converged for r in res)}/{len(res)}",
            "latency_ms": {"p50": 1e3 * float(np.percentile(lat, 50)), "p99": 1e3 * float(np.percentile(lat, 99))},
            "kernel_ms": prof,
            "roofline": {"bound": "hbm", "kernel": "CG step (A^ p, r1 update, A^T r1 over the matrix in pieces, column finish: four launches)",
                         "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS,
                         "traffic": None, "algorithmic_bytes_per_launch": alg_bytes}}


def _serve_leg(P, probs, arrivals=None, window=0):
    """Run the requests through one serving engine: open loop (request i is
    due at arrivals[i] seconds) or closed loop (at most ``window`` requests
    outstanding).  Latency runs from the due time (open) or the submit time
    (closed) to the poll that returns the result."""
    eng = P.BatchEngine(chunk_iters=25)
    try:
        start = time.perf_counter()
        pending, lat, statuses = {}, [], []
        i = 0
        while i < len(probs) or pending:
            now = time.perf_counter() - start
            if arrivals is not None:
                while i < len(probs) and arrivals[i] <= now:
                    pending[eng.submit(probs[i])] = arrivals[i]
                    i += 1
            else:
                while i < len(probs) and len(pending) < window:
                    pending[eng.submit(probs[i])] = time.perf_counter() - start
                    i += 1
            for tk in list(pending):
                r = eng.poll(tk)
                if r is not None:
                    lat.append(time.perf_counter() - start - pending.pop(tk))
                    statuses.append(r.status)
            time.sleep(0.0005)
        wall = time.perf_counter() - start
    finally:
        eng.close()
    conv = sum(s == P.POGS_CONVERGED for s in statuses)
    return {"solves_per_s": conv / wall, "wall_s": wall, "converged": f"{conv}/{len(statuses)}",
            "p50_ms": 1e3 * float(np.percentile(lat, 50)), "p99_ms": 1e3 * float(np.percentile(lat, 99))}


def bench_serve(args):
    """Mixed Lasso/NNLS/SVM/LP requests into the serving engine: the closed-loop
    maximum (``--window`` requests outstanding), then Poisson arrivals at 50 %
    and 80 % of it (p50/p99 latency), against the same requests solved one at
    a time on the whole-GPU path.  ``--qps`` > 0 adds one open-loop run at that
    rate."""
    from paper_1503_08366_amd import pogs as P
    from paper_1503_08366_amd import workloads as W
    block = serve_block(P, W, args.count, args.window, [0.5, 0.8], args.qps)
    return {"metric": "served solves/s at rel tol 1e-3 (continuous batching, closed loop) with p50/p99 latency "
                      "at 50%/80% of it (open loop)",
            "value": block["solves_per_s"], "unit": "solves/s", "n_gpus": 1, "higher_is_better": True,
            "config": {"workload": block["workload"], "window": args.window}, **block}


def serve_block(P, W, count, window, loads, qps=0.0):
    stream = list(W.serving_stream(count, 1.0))  # unit-rate arrivals; the problems do not depend on the rate
    unit = [t for t, _ in stream]
    probs = [p for _, p in stream]
    say = lambda msg: print(msg, file=sys.stderr, flush=True)
    # warm with one full leg: the device pool grows for every request size
    # once (the batch leg is warmed the same way)
    _serve_leg(P, probs, window=window)
    closed = _serve_leg(P, probs, window=window)
    say(f"serve closed loop: {closed}")
    t = time.perf_counter()
    plain_conv = 0
    prm = P.default_params(autotune=0)
    for p in probs:
        with P.Context(p.A, prm) as ctx:
            plain_conv += ctx.solve(p.f, p.g, prm).converged
    tp = time.perf_counter() - t
    say(f"serve plain: {plain_conv / tp:.1f} solves/s")
    rates = [f * closed["solves_per_s"] for f in loads] + ([qps] if qps > 0 else [])
    open_loop = []
    for q in rates:
        r = _serve_leg(P, probs, arrivals=[u / q for u in unit])
        r["offered_qps"] = q
        open_loop.append(r)
        say(f"serve open loop at {q:.1f}/s: {r}")
    last = open_loop[-1] if not qps else open_loop[len(loads) - 1]
    return {"workload": f"{count} requests, Lasso/NNLS/SVM/LP, m~logU[100,50000], n~logU[50,5000], "
                        "float32 host inputs (PCIe copy inside), HBM budget 80% of free",
            "solves_per_s": closed["solves_per_s"], "closed_loop": closed, "open_loop": open_loop,
            "latency_ms": {"p50": last["p50_ms"], "p99": last["p99_ms"], "at_qps": last["offered_qps"]},
            "plain": {"solves_per_s": plain_conv / tp, "seconds": tp, "converged": f"{plain_conv}/{len(probs)}",
                      "autotune": 0},
            "speedup": closed["solves_per_s"] / max(plain_conv / tp, 1e-30)}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="lasso", choices=sorted(WORKLOADS) + ["batch", "path", "serve", "sparse"])
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle leg")
    ap.add_argument("--no-blocks", action="store_true",
                    help="lasso: only the single-problem line (no dose, batched, path, serving blocks)")
    ap.add_argument("--serve-count", type=int, default=128, help="requests in the default line's serving block")
    ap.add_argument("--profile-reps", type=int, default=100)
    ap.add_argument("--count", type=int, default=512, help="batch / serve: number of problems")
    ap.add_argument("--plain-count", type=int, default=512, help="batch: problems in the plain leg")
    ap.add_argument("--R", type=int, default=64, help="path: number of lambdas")
    ap.add_argument("--qps", type=float, default=0.0, help="serve: one more open-loop run at this arrival rate")
    ap.add_argument("--window", type=int, default=128, help="serve: requests outstanding in the closed loop")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="MB",
                    help="only copy MB megabytes device-to-device three times (calibrates the HBM "
                         "byte counters against a plain copy of known size)")
    args = ap.parse_args()
    if args.copy_probe:
        import torch
        n = args.copy_probe * (1 << 20) // 4
        src = torch.ones(n, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_probe_bytes": 4 * n, "copies": 3}), flush=True)
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}); a multi-GPU sharding "
              "of the path is designed but not built", file=sys.stderr)
        sys.exit(2)
    if args.workload in ("batch", "path", "serve", "sparse"):
        import torch
        torch.cuda.set_device(0)
        out = {"batch": bench_batch, "path": bench_path, "serve": bench_serve,
               "sparse": bench_sparse}[args.workload](args)
        print(json.dumps(out), flush=True)
        return

    import torch
    from paper_1503_08366_amd import pogs as P
    from paper_1503_08366_amd import workloads as W
    torch.cuda.set_device(0)
    say = lambda msg: print(msg, file=sys.stderr, flush=True)

    line = single_problem(P, W, args.workload, args.steps, args.warmup, args.profile_reps, host_leg=True)
    prob_desc = line.pop("_prob")
    line = {
        "metric": "solves/s at rel tol 1e-3 (plain, one problem per launch sequence; batched, lambda-path and "
                  "served blocks beside it); ADMM iter/s; p50/p99 latency",
        **line}
    if not args.no_cpu:
        cb = cpu_baseline(prob_desc, projection=WORKLOADS[args.workload][2])
        line["cpu_baseline"] = cb
        line["oracle_rel_err"] = {args.workload: rel_err(line.pop("_optval"), cb["optval"])}
    else:
        line.pop("_optval")
    say(f"{args.workload}: {line['value']:.1f} solves/s")
    if args.workload == "lasso" and not args.no_blocks:
        # the metric's other workloads, each against its plain one-problem path
        dose = single_problem(P, W, "dose", 2, 1, 20, host_leg=False)
        dprob = dose.pop("_prob")
        drec = stored_oracle("dose_100000x1000.json", [dprob])
        dose["oracle_rel_err"] = None if drec is None else rel_err(dose.pop("_optval"), drec[0]["optval"])
        dose.pop("_optval", None)
        for k in ("metric", "n_gpus", "scaling", "vs_baseline", "data", "higher_is_better"):
            dose.pop(k, None)
        line["dose"] = dose
        say(f"dose: {dose['value']:.2f} solves/s")
        line["batched"] = batch_block(P, W.batch_mix(512), 512)
        say(f"batched: {line['batched']['solves_per_s']:.0f} solves/s, {line['batched']['speedup']:.2f}x plain")
        line["path"] = path_block(P, W.lambda_path())
        say(f"path: {line['path']['solves_per_s']:.0f} solves/s, {line['path']['speedup']:.2f}x plain")
        line["serving"] = serve_block(P, W, args.serve_count, min(args.window, args.serve_count), [0.8])
        say(f"serving: {line['serving']['solves_per_s']:.0f} solves/s")
    print(json.dumps(line), flush=True)


def single_problem(P, W, workload, steps, warmup, profile_reps, host_leg):
    """Whole solves of one problem with A resident in HBM (pogs_init + pogs_solve
    + pogs_free per step), the roofline of the dominant per-iteration kernel
    from HIP-event timings on the library's stream, and optionally the same
    solves from a host matrix (PCIe copy inside the timed region)."""
    import torch
    gen_name, desc, projection = WORKLOADS[workload]
    prob = getattr(W, gen_name)()
    m, n = prob.m, prob.n
    A = torch.from_numpy(prob.A).cuda()
    stream = torch.cuda.current_stream()
    prm = P.default_params(eps_abs=prob.eps_abs, eps_rel=prob.eps_rel, max_iter=prob.max_iter,
                           projection=projection)
    cgls = projection == "cgls"

    def step():
        t = time.perf_counter()
        with P.Context(A, prm, stream) as ctx:
            r = ctx.solve(prob.f, prob.g, prm, device_out=True)
        return time.perf_counter() - t, r

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    lat, res = [], []
    t0 = time.perf_counter()
    for _ in range(steps):
        dt, r = step()
        lat.append(dt)
        res.append(r)
    torch.cuda.synchronize()
    total = time.perf_counter() - t0
    converged = sum(r.converged for r in res)
    iters = sum(r.iters for r in res)
    solve_ms = sum(r.ms_solve for r in res)
    setup_ms = sum(r.ms_setup for r in res)

    host = None
    if host_leg:
        # the same whole solves with A handed over in (pageable) host memory: the
        # PCIe copy is inside the timed region
        host_steps = max(1, min(steps, 5))
        t = time.perf_counter()
        host_conv = 0
        for _ in range(host_steps):
            with P.Context(prob.A, prm, stream) as ctx:
                host_conv += ctx.solve(prob.f, prob.g, prm, device_out=True).converged
        torch.cuda.synchronize()
        host_s = time.perf_counter() - t
        host = {"solves_per_s": host_conv / host_s, "steps": host_steps,
                "input": "A in pageable host memory, PCIe copy inside the timed region"}

    # dominant kernel: the passes over A, timed with HIP events on the library's stream
    with P.Context(A, prm, stream) as ctx:
        ctx.solve(prob.f, prob.g, prm, device_out=True)
        prof = ctx.profile_iteration(profile_reps)
    del A
    tall = m >= n
    q = min(m, n)
    if cgls:
        # one CG step: A^ s (rows) and A^T [r1, q] (columns) plus the vectors
        kern = "cg_step"
        # tall float32 rows of at most 2048 entries: both products on one read of A
        once = tall and prob.A.dtype == np.float32 and n <= 2048
        alg_bytes = (4.0 if once else 8.0) * m * n + 4.0 * (5 * m + 8 * n)
        kern_desc = ("CG step (A p and A^T [r1, q] on one read of A, column finish: two launches)" if once
                     else "CG step (A p, A^T [r1, q]: three launches)")
        iter_bytes = None
        iter_bytes_read_once = None
    else:
        # one pass over A per iteration (tall float32): the prox step runs in
        # the first kernels, the profile reports no separate prox launch
        one_pass = tall and prof["prox"] == 0.0 and prob.A.dtype == np.float32 and n <= 2048
        vec_bytes = {  # vectors read + written per launch (float32, f64 column sums)
            "pass1": (2 * m + 3 * n) * 4 if tall else (2 * n + 3 * m) * 4,
            "pass2": (2 * n + 4 * m) * 4 if tall else (2 * m + 4 * n) * 4,
        }
        if one_pass:
            # reads x, x_h, d, y_h and f's five parameters and kind byte; writes
            # y, y~ and the next y_h, nu_h, d; the two column sums in float64
            vec_bytes["pass2"] = 4 * (2 * n + 7 * m) + m + 4 * 5 * m + 8 * 2 * n
        kern = max(("pass1", "pass2"), key=lambda k: prof[k])
        alg_bytes = 4.0 * m * n + vec_bytes[kern]
        if one_pass and kern == "pass2":
            kern_desc = "one-pass iteration kernel (y = A x, A x_h, next y-side half step, A^T [d', nu_h'])"
        else:
            kern_desc = f"{kern} ({'A^T v' if (kern == 'pass1') == tall else 'A v'})"
        # the method's bytes per iteration: two products with A, K^-1 and the vectors
        iter_bytes = 8.0 * m * n + 4.0 * q * q + 4.0 * 24 * (m + n)
        # what the one-pass iteration has to move: A once, K^-1, the vectors
        iter_bytes_read_once = 4.0 * m * n + 4.0 * q * q + 4.0 * 24 * (m + n) if one_pass else None
    achieved = alg_bytes / (prof[kern] * 1e-3) / 1e9
    traffic = None if cgls else recorded_traffic(workload, kern)
    line = {
        "value": converged / total,
        "unit": "solves/s",
        "n_gpus": 1,
        "steps": steps,
        "warmup": warmup,
        "ms_per_step": 1e3 * total / steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32 (f64 Gram reduction/Cholesky/norms)",
        "data": "synthetic (seeded, shaped as the paper's Lasso/NNLS/dose workloads)",
        "config": {"workload": desc, "m": m, "n": n, "eps_abs": prob.eps_abs, "eps_rel": prob.eps_rel,
                   "input": "A resident in HBM (torch tensor); outputs left on the device"},
        "admm_iter_per_s": iters / (solve_ms * 1e-3),
        "iters_per_solve": iters / len(res),
        "converged": f"{converged}/{len(res)}",
        "setup_ms_mean": setup_ms / len(res),
        "solve_ms_mean": solve_ms / len(res),
        "latency_ms": {"p50": 1e3 * float(np.percentile(lat, 50)), "p99": 1e3 * float(np.percentile(lat, 99))},
        "kernel_ms": prof,
        "roofline": {"bound": "hbm", "kernel": kern_desc,
                     "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                     "algorithmic_bytes_per_launch": alg_bytes},
        "_optval": float(res[-1].optval),
        "_prob": prob,
    }
    if host is not None:
        line["host_input"] = host
    if iter_bytes is not None:
        # iteration_GBps / iteration_frac: the method's bytes per iteration
        # (both products with A) over the measured iteration time
        line["iteration_GBps"] = iter_bytes / (prof["iteration"] * 1e-3) / 1e9
        line["iteration_frac"] = line["iteration_GBps"] / HBM_PEAK_GBS
        if iter_bytes_read_once is not None:
            line["iteration_moved_GBps"] = iter_bytes_read_once / (prof["iteration"] * 1e-3) / 1e9
            line["iteration_moved_frac"] = line["iteration_moved_GBps"] / HBM_PEAK_GBS
            line["iteration_note"] = ("A is read once per iteration (both products from one read), so the "
                                      "method's two-pass bytes over the time exceed what moves; "
                                      "iteration_moved_* counts A once")
    if cgls:
        line["cg_steps_per_iteration"] = sum(r.cg_steps for r in res) / max(iters, 1)
    return line


if __name__ == "__main__":
    main()
