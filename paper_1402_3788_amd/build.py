"""Build libkmeans_mi355x.so (the HIP library behind include/kmeans.h) in-tree.

Usage: python paper_1402_3788_amd/build.py
(run as a script: importing the package needs the library this builds)
"""
from __future__ import annotations

import os
import subprocess
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libkmeans_mi355x.so")
# Flags of one translation unit: the small-K kernel is scheduled with the
# compiler's iterative scheduler aiming at occupancy (measured per launch at
# n = 2e6, M = 25, K = 16: 38.2 us against 39.1 with the default scheduler and
# 38.9 with the instruction-level-parallelism one; the same as the default at
# K = 64 on 2e7 objects; the tile kernel is slower with any of them); the L1
# assignment kernel for instruction-level parallelism (an L1 iteration at
# K = 16: 99.7 us against 103.4 with the default scheduler); the direct-form
# lane kernel likewise (at n = 2e6, M = 25, K = 16: a fused L1 iteration
# 66.2-66.6 us against 69.3-69.4, a direct-form Euclidean iteration 64.2-64.3
# against 65.7-65.9).
UNIT_FLAGS = {"lloyd_lane_mfma.hip": ["-mllvm", "-amdgpu-sched-strategy=iterative-maxocc"],
              "lloyd_l1.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"],
              "lloyd_lane.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]}
# (source, extra flags, object name); the kernel files are compiled once per
# part of the feature-count range so the template instantiations build in parallel
PARTS = 4
SOURCES = ([("kmeans_api.hip", [], "kmeans_api.o"), ("lloyd_ctl.hip", [], "lloyd_ctl.o"),
            ("lloyd_centres.hip", [], "lloyd_centres.o"), ("farthest.hip", [], "farthest.o"),
            ("lloyd_accum.hip", [], "lloyd_accum.o"),
            ("diameter.hip", [], "diameter.o"), ("lloyd_l1.hip", UNIT_FLAGS["lloyd_l1.hip"], "lloyd_l1.o")]
           + [(f, [f"-DLLOYD_PART={p}", *UNIT_FLAGS.get(f, [])], f.replace(".hip", f"_part{p}.o"))
              for f in ("lloyd_tile.hip", "lloyd_lane.hip", "lloyd_lane_mfma.hip")
              for p in range(PARTS)])
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # every floating-point operation is rounded on its own unless written as
    # an explicit fma; the fp64 tie re-check relies on it
    "-ffp-contract=off",
    # keep the compiler from forming packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def _newest_header() -> float:
    heads = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    heads.append(os.path.join(ROOT, "include", "kmeans.h"))
    return max(os.path.getmtime(h) for h in heads)


def build(verbose: bool = True, jobs: int = 8, incremental: bool = False) -> str:
    """Compile every source to an object file (in parallel), then link.
    incremental: skip objects newer than their source and every header."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    t0 = time.time()
    head_t = _newest_header()
    for src, extra, oname in SOURCES:
        obj = os.path.join(objdir, oname)
        objs.append(obj)
        if incremental and os.path.exists(obj):
            ot = os.path.getmtime(obj)
            if ot > os.path.getmtime(os.path.join(CSRC, src)) and ot > head_t:
                continue
        cmd = [hipcc(), *HIPCC_FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            time.sleep(0.05)
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        text = out.decode(errors="replace")
        if p.returncode != 0:
            failed = True
            sys.stderr.write(f"--- {src} failed ---\n{text}\n")
        elif verbose and text.strip():
            # the host pass does not know the packed-fp32 feature name; skip that note
            lines = [ln for ln in text.splitlines() if "packed-fp32-ops" not in ln]
            if lines:
                sys.stderr.write("\n".join(lines) + "\n")
    if failed:
        raise RuntimeError("HIP compilation failed")
    tmp = LIB + ".tmp"
    subprocess.check_call([hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB} in {time.time() - t0:.1f}s")
    return LIB


if __name__ == "__main__":
    build(incremental="--incremental" in sys.argv)
