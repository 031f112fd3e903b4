"""Build liblbm.so (HIP, gfx950) in-tree with hipcc.

Usage: python -m paper_1203_6350_amd.build  (or paper_1203_6350_amd.build.build())
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "liblbm.so")
# (source, extra flags, object name): the strip kernels compile once per
# step count K, so that the largest translation units build side by side
SOURCES = [(f, [], f.rsplit(".", 1)[0]) for f in
           ("lbm_api.cpp", "lbm_kernels.hip", "lbm_vn.hip", "lbm_batch.hip", "lbm3_kernels.hip",
            "lbm_readout.cpp")]
SOURCES += [("lbm_strip_%s.hip" % st, ["-DLBM_STRIP_ONLY_K=%d" % k], "lbm_strip_%s_k%d" % (st, k))
            for st in ("f32", "f64", "f16") for k in (6, 5, 4, 3, 2)
            if k <= {"f32": 6, "f64": 5, "f16": 4}[st]]
SOURCES += [("lbm_tile_%s.hip" % st, [], "lbm_tile_%s" % st) for st in ("f32", "f64", "f16")]

# - no automatic FMA contraction: the kernels place their fused multiply-adds
#   explicitly, so every launch shape gives the same bits;
# - packed FP32 instructions disabled for all device code.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False, jobs: int | None = None) -> str:
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    cc = hipcc()
    cmds, objs = [], []
    for src, extra, name in SOURCES:
        obj = os.path.join(bdir, name + ".o")
        cmds.append([cc, "-x", "hip"] + [f for f in FLAGS if f != "-shared"] + extra + [
            "-I", os.path.join(ROOT, "include"), "-c", os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    # the translation units are independent: compile them side by side
    jobs = jobs or max(1, min(len(cmds), os.cpu_count() or 1, 8))
    procs = []
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        while len([p for p in procs if p.poll() is None]) >= jobs:
            time.sleep(0.2)
        procs.append(subprocess.Popen(cmd))
    failed = [c for c, p in zip(cmds, procs) if p.wait() != 0]
    if failed:
        raise subprocess.CalledProcessError(1, failed[0])
    tmp = OUT + ".tmp%d" % os.getpid()
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
