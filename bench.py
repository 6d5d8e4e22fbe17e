"""Benchmark: Lloyd iterations per second on one MI355X.

A step is one Lloyd iteration of Algorithm 1 over the whole point set: a
launch that assigns every object (steps 2/4) and accumulates the sums of
Eq. (1) per workgroup, then a small launch that forms the new centres from
those partials and compares them with the previous ones (steps 6/7).
The default workload is the paper's largest size: n = 2,000,000 objects,
M = 25 features, K = 16 clusters (anisotropic Gaussian blobs, seed 2,
farthest-point initial centres). Iterations run in fixed-count mode so every
timed step does the full work (this workload converges after 2 passes; the
passes after that repeat the same labels and centres). X is resident in device
memory before the timed region starts.

The JSON line also times the paper's own stopping rule (a call that runs until
the centres are congruent, "converge_mode"), and, on the same workload, the
farthest-point initial
centres of Algorithm 1 step 1 (K passes over X, "init_farthest") and the
diameter of Eq. (3) with the centre of gravity (Algorithm 2 steps 1-2, two
passes over all pairs on the fp16 matrix cores, "diameter"), and Lloyd
iterations that assign by the L1 distance instead ("l1_metric").

python bench.py [--gpus 1] [--steps 1000] [--warmup 20] [--workload 3]
                [--path auto|direct|mfma|tiles] [--no-cpu-baseline] [--no-control]
                [--no-init] [--no-diameter] [--no-l1]
python bench.py --calibrate-copy   # plain device copy of known size (PMC scaling)

Prints ONE JSON line.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import re
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0          # MI355X HBM3E, vendor peak
PROFILES = os.path.join(ROOT, "profiles")
CSRC = os.path.join(ROOT, "paper_1402_3788_amd", "csrc")
METRIC = "Lloyd iters/sec and points·iters/sec at n=2e6,M=25,K=16; % of HBM peak"
PROTOCOL_RUNS = 10          # calls timed with events before the timed region
PROTOCOL_ITERS = 100        # iterations per such call (iteration time)
PROTOCOL_KERNEL_ITERS = 20  # iterations per call with every assign launch timed

# arithmetic of the distance step on each path (the sums are fp64 on all)
DTYPE = {"lane-mfma": "bf16x3-split/f32-acc, f64 re-decision", "tiles": "bf16x3-split/f32-acc, f64 re-decision",
         "direct": "f32, f64 re-decision"}
DISTANCE = {
    "lane-mfma": "expanded form on the bf16 matrix cores: operands split into bf16 hi and lo, "
                 "three products per block, fp32 accumulation; close calls re-decided in fp32 direct form or fp64",
    "tiles": "expanded form on the bf16 matrix cores: operands split into bf16 hi and lo, "
             "up to three products per block, fp32 accumulation; close calls re-decided "
             "in fp64 among their candidates",
    "direct": "direct form in fp32 on the vector ALU; close calls re-decided in fp64",
}

# kernel that does the work of a step on each distance path, and the sources
# it is built from (a committed counter summary is used only while they match)
KERNELS = {
    "lane-mfma": ("lane_mfma_kernel<M, assign+accumulate> (split bf16 products)",
                  ["lloyd_lane_mfma.hip", "lloyd_device.h", "lloyd.h"]),
    "direct": ("lloyd_lane_kernel<M, assign+accumulate, P>",
               ["lloyd_lane.hip", "lloyd_device.h", "lloyd.h"]),
    "tiles": ("lloyd_tile_kernel<M, assign+accumulate, acc>",
              ["lloyd_tile.hip", "lloyd_device.h", "lloyd.h"]),
}


def _parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1000)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="3")
    ap.add_argument("--path", default="auto", choices=["auto", "direct", "mfma", "tiles"])
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-control", action="store_true")
    ap.add_argument("--no-init", action="store_true")
    ap.add_argument("--no-diameter", action="store_true")
    ap.add_argument("--no-l1", action="store_true")
    ap.add_argument("--calibrate-copy", action="store_true")
    return ap.parse_args()


def kernel_key(M: int, K: int, path: str) -> str:
    """Which kernel runs the iteration (mirrors the library's path choice)."""
    lane_fits = K <= 64 and M <= 32
    if path == "direct":
        return "direct"
    if path == "tiles":
        return "tiles"
    if path == "mfma":
        return "lane-mfma" if lane_fits else "tiles"
    if lane_fits and K >= 5:
        return "lane-mfma"
    return "tiles" if K > 16 else "direct"


def sources_sha256(key: str) -> str:
    h = hashlib.sha256()
    for name in KERNELS[key][1]:
        with open(os.path.join(CSRC, name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def _traffic(key: str, workload: str):
    """HBM bytes per launch from the committed counter summary for this kernel
    and workload, if it was taken on the current sources; else None."""
    path = os.path.join(PROFILES, f"pmc_{key}_{workload}.md")
    if not os.path.exists(path):
        return None
    m = re.search(r"```json\n(.*?)\n```", open(path).read(), re.S)
    if not m:
        return None
    d = json.loads(m.group(1))
    if d.get("sources_sha256") != sources_sha256(key):
        return None
    return d.get("hbm_bytes_per_launch")


def calibrate_copy():
    import torch
    n = 1 << 28                                   # 2^28 fp32 = 1 GiB
    src = torch.ones(n, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    for _ in range(10):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes_read": 4 * n, "copy_bytes_written": 4 * n, "launches": 10}))


def copy_bandwidth(torch, nbytes=1 << 30, reps=20):
    n = nbytes // 4
    src = torch.ones(n, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    dst.copy_(src)
    s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    s.record()
    for _ in range(reps):
        dst.copy_(src)
    e.record()
    torch.cuda.synchronize()
    sec = s.elapsed_time(e) / 1e3 / reps
    del src, dst
    return 2 * nbytes / sec / 1e9


def host_info() -> dict:
    """CPU model and logical CPU count of the host this runs on."""
    model = None
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"cpu_model": model, "nproc": os.cpu_count()}


def init_bytes(n: int, M: int, K: int) -> int:
    """Algorithmic bytes of the farthest-point traversal: pass p = 1 .. K-1
    reads X, reads the fp64 nearest distances (p > 1) and writes them (when a
    later pass reads them)."""
    return sum(n * 4 * M + (8 * n if p > 1 else 0) + (8 * n if p + 1 < K else 0)
               for p in range(1, K))


def time_init(torch, km, Xg, K, stored, reps=5):
    n, M = Xg.shape
    ws = torch.empty(km.kmeans_init_workspace_bytes(n, M, K), dtype=torch.uint8,
                     device=Xg.device)
    idx, _ = km.kmeans_init_farthest(Xg, K, ws=ws)             # warm-up, and a check
    torch.cuda.synchronize()
    same = bool((idx.cpu().numpy() == stored).all())
    s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    s.record()
    for _ in range(reps):
        km.kmeans_init_farthest(Xg, K, ws=ws)
    e.record()
    torch.cuda.synchronize()
    sec = s.elapsed_time(e) / 1e3 / reps
    nbytes = init_bytes(n, M, K)
    return {
        "ms": round(sec * 1e3, 3),
        "launches": K,
        "bytes": nbytes,
        "achieved_GBps": round(nbytes / sec / 1e9, 1) if K > 1 else None,
        "frac_hbm_peak": round(nbytes / sec / 1e9 / HBM_PEAK_GBPS, 4) if K > 1 else None,
        "matches_stored_init": same,
        "reps": reps,
    }


BF16_PEAK_TFLOPS = 2500.0       # MI355X dense bf16 (and fp16) matrix peak


def time_diameter(torch, km, Xg, reps=2):
    """Priced as one screening pass over the n(n-1)/2 pairs: one fp16 matrix product
    over 32 ceil((M+2)/32) features per pair (the second pass only
    revisits the few work items whose maximum reaches the threshold)."""
    n, M = Xg.shape
    ws = torch.empty(km.kmeans_diameter_workspace_bytes(n, M), dtype=torch.uint8,
                     device=Xg.device)
    d2a, paira, _ = km.kmeans_diameter(Xg, ws=ws)             # warm-up
    torch.cuda.synchronize()
    s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    s.record()
    for _ in range(reps):
        d2, pair, _ = km.kmeans_diameter(Xg, ws=ws)
    e.record()
    torch.cuda.synchronize()
    sec = s.elapsed_time(e) / 1e3 / reps
    P = 32 * ((M + 2 + 31) // 32)
    pairs = n * (n - 1) // 2
    flops = pairs * 2 * P
    return {
        "ms": round(sec * 1e3, 2),
        "d2": float(d2.item()),
        "pair": [int(v) for v in pair.cpu().numpy()],
        "repeatable": bool(d2.item() == d2a.item() and torch.equal(pair, paira)),
        "pairs_per_s": round(pairs / sec, 1),
        "fp16_matrix_TFLOPs": round(flops / sec / 1e12, 1),
        "frac_fp16_peak": round(flops / sec / 1e12 / BF16_PEAK_TFLOPS, 4),
        "reps": reps,
    }


def main():
    args = _parse()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); "
              "sharding the Lloyd iteration over several GPUs (one all-gather of the fp64 "
              "partial sums per iteration) is designed but not built", file=sys.stderr)
        sys.exit(2)
    if args.calibrate_copy:
        calibrate_copy()
        return

    import numpy as np
    import torch

    import paper_1402_3788_amd as km
    import workloads

    w = workloads.get(args.workload)
    X, _, init_idx, init = workloads.load(args.workload)
    dev = torch.device("cuda:0")
    Xg = torch.from_numpy(X).to(dev)
    Cg = torch.from_numpy(init).to(dev)
    n, M, K = w.n, w.M, w.K
    path = None if args.path == "auto" else args.path
    key = kernel_key(M, K, args.path)
    flags = km._flags(path) | km.KMEANS_FIXED_ITERS
    out = (torch.empty(n, dtype=torch.int32, device=dev),
           torch.empty((K, M), dtype=torch.float32, device=dev),
           torch.empty(K, dtype=torch.int32, device=dev))
    ws = km.workspace(n, M, K, dev, flags)

    # Kernel and iteration times from HIP events of the library's own: on
    # the launch stream, PROTOCOL_RUNS fixed-count calls of PROTOCOL_ITERS
    # iterations with events around every call, and PROTOCOL_RUNS calls whose
    # every assign + accumulate launch is made with a pair of events that its
    # dispatch stamps at start and end (the kernel's own duration, as a kernel
    # trace reports it); medians over the calls.
    # They run before the timed region, which they also bring out of the
    # idle state (low clocks) the input generation left the GPU in.
    it_us, k_us = [], []
    nsamp = 0
    for _ in range(PROTOCOL_RUNS):
        # events only around the call (and the first launch): iteration time
        _, _, _, _, tm = km.kmeans_run(Xg, K, Cg, PROTOCOL_ITERS, fixed_iters=True, path=path,
                                       timing=True, sample_every=PROTOCOL_ITERS + 1, out=out,
                                       ws=ws)
        it_us.append(tm.step_ms * 1e3 / tm.step_launches)
    for _ in range(PROTOCOL_RUNS):
        # every assign + accumulate launch stamped by its dispatch: the kernel's duration
        _, _, _, _, tm = km.kmeans_run(Xg, K, Cg, PROTOCOL_KERNEL_ITERS, fixed_iters=True,
                                       path=path, timing=True, sample_every=1, out=out, ws=ws)
        k_us.append(tm.assign_ms * 1e3 / tm.assign_samples)
        nsamp += tm.assign_samples
    # warmup
    km.kmeans_run(Xg, K, Cg, max(1, args.warmup), fixed_iters=True, path=path, out=out, ws=ws)
    torch.cuda.synchronize()

    # timed region: exactly `steps` Lloyd iterations in one fixed-count call,
    # host clock, bracketed by device synchronisation; no events inside it
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    _, _, _, iters = km.kmeans_run(Xg, K, Cg, args.steps, fixed_iters=True, path=path,
                                   out=out, ws=ws)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    assert iters == args.steps
    sec = t1 - t0
    iters_per_s = args.steps / sec
    fallbacks = km.ctl_fallbacks(ws)
    reruns = km.ctl_reruns(ws)
    bytes_per_point = 4 * M + 4                    # read the object once, write its label
    launch_bytes = n * bytes_per_point

    iteration_us = statistics.median(it_us)
    assign_us = statistics.median(k_us)
    achieved = launch_bytes / (assign_us * 1e-6) / 1e9
    traffic = _traffic(key, w.name)

    result = {
        "metric": METRIC,
        "value": round(iters_per_s, 2),
        "unit": "iters/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(sec * 1e3 / args.steps, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": DTYPE.get(key, "f32"),
        "data": "synthetic",
        "config": {"workload": w.name, "n": n, "M": M, "K": K, "mode": "fixed iterations",
                   "distance": DISTANCE.get(key), "accumulation": "f64 sums in a fixed order",
                   "path": args.path},
        "points_iters_per_s": round(iters_per_s * n, 1),
        "algorithmic_GBps_whole_step": round(launch_bytes * iters_per_s / 1e9, 1),
        "pct_hbm_peak_whole_step": round(100 * launch_bytes * iters_per_s / 1e9 / HBM_PEAK_GBPS, 2),
        # the protocol runs (events on the launch stream, medians over the calls)
        "protocol": {"calls": PROTOCOL_RUNS, "iterations_per_call": PROTOCOL_ITERS,
                     "kernel_calls": PROTOCOL_RUNS,
                     "kernel_iterations_per_call": PROTOCOL_KERNEL_ITERS,
                     "iteration_median_us": round(iteration_us, 3),
                     "iteration_min_us": round(min(it_us), 3),
                     "iteration_max_us": round(max(it_us), 3),
                     "assign_launch_median_us": round(assign_us, 3),
                     "assign_launches_timed": nsamp},
        "kernel_avg_us": round(assign_us, 3),
        "iteration_avg_us": round(iteration_us, 3),
        # close calls of the timed run, per iteration: columns of up to 16
        # objects scored again (tile kernel), objects decided again (both
        # kernels)
        "reruns_per_iteration": round(reruns / args.steps, 2),
        "fallbacks_per_iteration": round(fallbacks / args.steps, 2),
        "roofline": {
            "bound": "hbm",
            "achieved": round(achieved, 1),
            "peak": HBM_PEAK_GBPS,
            "unit": "GB/s",
            "frac": round(achieved / HBM_PEAK_GBPS, 4),
            "traffic": traffic,
            "kernel": KERNELS[key][0].replace("<M,", f"<{M},"),
            "bytes_per_launch": launch_bytes,
            "launch_us": round(assign_us, 3),
        },
    }

    if key == "tiles":
        # the 64-object-tile kernel is matrix-bound for large K: it issues three
        # bf16 products per 16 x 16 block of (object, centre) pairs and 32
        # features, two (one) for a last chunk of at most 16 (8) features
        last = M - 32 * (-(-M // 32) - 1)
        products = 3 * (-(-M // 32) - 1) + (1 if last <= 8 else 2 if last <= 16 else 3)
        flops = products * 2 * (64 * -(-n // 64)) * (16 * -(-K // 16)) * 32
        tf = flops / (assign_us * 1e-6) / 1e12
        result["roofline_mfma"] = {"bound": "mfma", "achieved": round(tf, 1),
                                   "peak": BF16_PEAK_TFLOPS, "unit": "TFLOP/s",
                                   "frac": round(tf / BF16_PEAK_TFLOPS, 4),
                                   "flops_per_launch": flops}

    # the paper's own stopping rule (centres congruent): end-to-end latency of
    # one synchronous call from the initial centres, host clock
    km.kmeans_run(Xg, K, Cg, w.max_iter, path=path, out=out, ws=ws)
    torch.cuda.synchronize()
    tc = time.perf_counter()
    _, _, _, conv_iters = km.kmeans_run(Xg, K, Cg, w.max_iter, path=path, out=out, ws=ws)
    conv_s = time.perf_counter() - tc
    result["converge_mode"] = {"iterations": conv_iters, "max_iter": w.max_iter,
                               "ms": round(conv_s * 1e3, 3)}

    if not args.no_init:
        result["init_farthest"] = time_init(torch, km, Xg, K, init_idx)

    if not args.no_diameter:
        result["diameter"] = time_diameter(torch, km, Xg)

    if not args.no_l1:
        # the other metric: the L1 assignment fused with the accumulation
        # where its per-wave slabs leave enough waves (else an L1 assign launch
        # and an accumulate-from-labels launch), then the centres launch
        T = 200
        ws = km.workspace(n, M, K, dev, km.KMEANS_FIXED_ITERS | km.KMEANS_METRIC_L1)
        km.kmeans_run(Xg, K, Cg, 5, fixed_iters=True, metric="l1", out=out, ws=ws)
        torch.cuda.synchronize()
        _, _, _, _, tml = km.kmeans_run(Xg, K, Cg, T, fixed_iters=True, metric="l1", timing=True,
                                        out=out, ws=ws)
        result["l1_metric"] = {
            "iters_per_s": round(T / (tml.step_ms / 1e3), 1),
            "iteration_avg_us": round(tml.step_ms * 1e3 / T, 2),
            "assign_launch_avg_us": round(tml.assign_ms * 1e3 / tml.assign_samples, 2),
            "fallbacks_per_iteration": round(km.ctl_fallbacks(ws) / T, 2),
            "steps": T,
        }

    if not args.no_control:
        # same kernel on a point set larger than the 256 MB Infinity Cache
        rng = np.random.default_rng(123)
        nc = 8_000_000
        Xc = torch.from_numpy(rng.uniform(-50, 50, (nc, M)).astype(np.float32)).to(dev)
        Cc = Xc[:K].clone()
        km.kmeans_run(Xc, K, Cc, 5, fixed_iters=True, path=path)
        wsc = km.workspace(nc, M, K, dev, flags)
        _, _, _, _, tmc = km.kmeans_run(Xc, K, Cc, 50, fixed_iters=True, path=path,
                                        timing=True, sample_every=1, ws=wsc)
        avg = tmc.assign_ms / 1e3 / tmc.assign_samples
        result["control_n8m_uniform"] = {
            "kernel_avg_us": round(avg * 1e6, 2),
            "achieved_GBps": round(nc * bytes_per_point / avg / 1e9, 1),
            # uniform objects sit near bisectors far more often than clustered
            # ones: the fp64 re-decisions are part of this launch's time
            "fallbacks_per_iteration": round(km.ctl_fallbacks(wsc) / 50, 1),
        }
        del Xc
        result["copy_GBps_torch_1GiB"] = round(copy_bandwidth(torch), 1)

    if not args.no_cpu_baseline:
        import oracle
        host = host_info()
        # the oracle is single-threaded; pin this process to one core while it
        # runs (in-process, no re-launch), then restore the affinity
        allowed = os.sched_getaffinity(0)
        core = min(allowed)
        os.sched_setaffinity(0, {core})
        try:
            t = time.perf_counter()
            oracle.run(X, K, init, 1, fixed=True)
            one = time.perf_counter() - t
            T = int(max(1, min(20, 15.0 // max(one, 1e-3))))
            t = time.perf_counter()
            oracle.run(X, K, init, T, fixed=True)
            cpu_s = time.perf_counter() - t
        finally:
            os.sched_setaffinity(0, allowed)
        result["cpu_baseline"] = {
            "value": round(T / cpu_s, 4),
            "unit": "iters/s",
            "cores": 1,
            "kind": "oracle",
            "sample": f"{T} fixed Lloyd iterations over all {n} objects of the same workload "
                      f"(single-threaded C, fp64), pinned to core {core}",
            "cpu_model": host["cpu_model"],
            "nproc": host["nproc"],
            "cores_available": len(allowed),
        }
        # the paper's multi-threaded CPU regime (Algorithm 3) on every host
        # thread OpenMP offers: a second baseline, not the oracle
        t = time.perf_counter()
        *_, used = oracle.alg3_run(X, K, init, 1, fixed=True)
        one = time.perf_counter() - t
        T = int(max(1, min(100, 10.0 // max(one, 1e-3))))
        t = time.perf_counter()
        oracle.alg3_run(X, K, init, T, fixed=True)
        alg3_s = time.perf_counter() - t
        result["cpu_baseline"]["alg3"] = {
            "value": round(T / alg3_s, 4),
            "unit": "iters/s",
            "cores": used,
            "kind": "Algorithm 3 (multi-threaded CPU regime, OpenMP, fp64)",
            "sample": f"{T} fixed Lloyd iterations over all {n} objects of the same workload",
        }
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
