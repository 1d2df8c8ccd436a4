"""Build the HIP library in-tree for gfx950 (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libschedsim.so")
SOURCES = [os.path.join(PKG, "csrc", f) for f in
           ("sched_wave_amin.hip", "sched_wave_aell.hip", "sched_wave_amax.hip", "sched_wave_hsf.hip",
            "sched_wave_arandom.hip", "sched_wide.hip", "sched_group.hip", "sched_group_amin.hip", "sched_kernels.hip",
            "opt_kernels.hip")]
HEADERS = [os.path.join(PKG, "csrc", "wave.hpp"), os.path.join(PKG, "csrc", "sim_device.hpp"),
           os.path.join(PKG, "csrc", "sim_wave.hpp"), os.path.join(PKG, "csrc", "sim_tiny.hpp"),
           os.path.join(PKG, "csrc", "prepare.hpp"),
           os.path.join(ROOT, "include", "schedsim.h")]
# throughput probes for the roofline (measurement infrastructure, own library)
PROBE_LIB = os.path.join(PKG, "libschedprobe.so")
PROBE_SOURCES = [os.path.join(PKG, "csrc", "probe_kernels.hip")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I" + os.path.join(ROOT, "include"),
]
# the one-wave kernels are in sched_wave_*.hip, one policy each
SPLIT_FLAGS = ["-DSK_SEPARATE_KERNELS"]
# The simulation kernels are latency-bound chains of dependent instructions on
# one wave; LLVM's iterative ILP scheduling strategy measured 1-7% faster than
# the default occupancy-first one on them (the probes keep the default).  Their
# step loops branch on uniform values only: without the structurizer's masks (it
# leaves uniform regions alone) and the flags that scope exits would set for the
# lifetime markers, such a branch is one scalar compare and jump.  Together with
# code written for it, 1.2 times faster over all policies.
SIM_FLAGS = ["-mllvm", "--amdgpu-sched-strategy=iterative-ilp", "-mllvm", "-structurizecfg-skip-uniform-regions"]
NO_MARKERS = ["-Xclang", "-disable-lifetime-markers"]
# The workgroup kernels other than A_min's keep the markers: without them one instance of
# 100000 on 4 waves took 272 ms instead of 250 (A_max) and 157 instead of 135 (H-SF), where
# A_min took 397 instead of 428.
KEEP_MARKERS = ("sched_group.hip",)


def _compile(sources, lib, verbose, extra, flags_of=lambda name: ()):
    """Each translation unit to an object (concurrently, in _build/), then one
    shared library (every object carries its own device code)."""
    objdir = os.path.join(ROOT, "_build")
    os.makedirs(objdir, exist_ok=True)
    tag = f"{os.getpid()}"
    objs, procs = [], []
    for src in sources:
        obj = os.path.join(objdir, os.path.basename(src) + f".{tag}.o")
        cmd = [HIPCC, *[f for f in FLAGS if f != "-shared"], *flags_of(os.path.basename(src)), *extra, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((subprocess.Popen(cmd), cmd))
        objs.append(obj)
    failed = [cmd for p, cmd in procs if p.wait() != 0]
    try:
        if failed:
            raise subprocess.CalledProcessError(1, failed[0])
        tmp = lib + f".tmp{tag}"
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp])
        os.replace(tmp, lib)
    finally:
        for obj in objs:
            if os.path.exists(obj):
                os.remove(obj)


def build(verbose: bool = True, extra=()) -> str:
    """Compile libschedsim.so and libschedprobe.so (always recompiles)."""
    _compile(SOURCES, LIB, verbose, [*SIM_FLAGS, *SPLIT_FLAGS, *extra],
             lambda name: () if name in KEEP_MARKERS else NO_MARKERS)
    _compile(PROBE_SOURCES, PROBE_LIB, verbose, extra)
    return LIB


if __name__ == "__main__":
    build(extra=sys.argv[1:])
