"""Build libh2mg.so (HIP for gfx950 + host C++) in-tree with hipcc.

Usage: python -m paper_2501_17656_amd.build   (or build() from Python).
Every call recompiles every source.
"""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libh2mg.so")

HIP_SOURCES = ["kernels_setup.hip", "kernels_apply.hip", "kernels_near.hip", "kernels_sweep.hip", "kernels_sweep16.hip",
               "kernels_solve.hip", "kernels_bem.hip",
               "kernels_block.hip", "noalloc.hip"]
CPP_SOURCES = ["plan.cpp", "h2_build.cpp", "h2_apply.cpp", "block.cpp", "solver.cpp", "abi.cpp"]
ARCH = os.environ.get("H2MG_ARCH", "gfx950")


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build the library)")


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), "-std=c++17", "-O3", "-fPIC", "-I", INCLUDE, "-I", CSRC, "-c",
           os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".hip"):
        cmd[1:1] = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops"]
    if src == "plan.cpp":
        # box tests must round like plain IEEE operations, one at a time
        cmd.insert(1, "-ffp-contract=off")
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compiling {src} failed:\n{res.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = HIP_SOURCES + CPP_SOURCES
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"linking libh2mg.so failed:\n{res.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
