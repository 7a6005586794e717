"""Builds libgp.so (the C-ABI library) in-tree with hipcc for gfx950.

    python -m paper_2207_12000_amd.build [--force]
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libgp.so")

SOURCES = ["gp_api.cpp", "gp_plan.cpp", "gp_schedule.cpp", "gp_cluster.cpp", "gp_propagate.cpp", "gp_stream.cpp", "gp_solve.cpp", "gp_kernels.hip", "gp_noalloc.hip", "gp_hot_lds.hip", "gp_device_sort.hip", "gp_plan_device.hip", "gp_cluster_device.hip", "gp_lc.hip", "gp_lc_f32.hip"]

COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          "-I", os.path.join(ROOT, "include"), "-I", CSRC]
# device code: gfx950 only; packed-fp32 instructions switched off
DEVICE = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def _stale(target: str, deps) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = False, verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    headers = [os.path.join(CSRC, "gp_internal.h"), os.path.join(CSRC, "gp_block_scan.h"), os.path.join(CSRC, "gp_lc.h"), os.path.join(ROOT, "include", "gp.h")]
    hipcc = _hipcc()

    def compile_one(name: str) -> str:
        src = os.path.join(CSRC, name)
        obj = os.path.join(OBJ, name + ".o")
        if force or _stale(obj, [src] + headers):
            cmd = [hipcc] + COMMON + DEVICE + ["-x", "hip", "-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    if force or _stale(LIB, objs):
        tmp = LIB + f".tmp{os.getpid()}"
        cmd = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs + ["-lpthread"]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    import argparse
    ap = argparse.ArgumentParser()
    ap.add_argument("--force", action="store_true")
    a = ap.parse_args()
    print(build(force=a.force, verbose=True))
