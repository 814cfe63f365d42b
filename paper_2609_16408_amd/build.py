"""Build the HIP shared library librpa_mi355x.so in-tree for gfx950.

Usage: python -m paper_2609_16408_amd.build [--verbose]
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB_NAME = "librpa_mi355x.so"
LIB_PATH = os.path.join(PKG, LIB_NAME)
SOURCES = ["engine.hip", "cocg.hip", "cocg_resident.hip", "kernels.hip", "transform.hip", "server.hip", "precond.hip",
           "block_lanczos.hip"]
# the persistent COCG kernels: one object per variant (plain, nonlocal,
# preconditioned, both) and LDS pitch
COCG_GROUPS = [(v, pitch) for v in (3, 2, 1, 0) for pitch in (56, 64, 128)]
ARCH = "gfx950"


def hipcc() -> str:
    for cand in ("/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def common_flags() -> list:
    return [
        "-O3", "-std=c++17", f"--offload-arch={ARCH}", "-fPIC",
        # no packed-FP32 instructions anywhere in the device code
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", INCLUDE, "-I", CSRC,
        "-Wno-unused-command-line-argument",
    ]


def _compile(src: str, verbose: bool, name: str = "", defines=()) -> str:
    obj = os.path.join(BUILD_DIR, (name or os.path.splitext(src)[0]) + ".o")
    cmd = [hipcc(), *common_flags(), *defines, "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{res.stderr}")
    if verbose and res.stderr.strip():
        print(res.stderr, flush=True)
    return obj


def build(verbose: bool = False) -> str:
    """Compile every HIP source and link the shared library; returns its path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    jobs = [("cocg_kernels.hip", f"cocg_v{v}_p{p}", (f"-DRPA_V={v}", f"-DRPA_PITCH={p}")) for v, p in COCG_GROUPS]
    jobs += [(s, "", ()) for s in SOURCES]
    with cf.ThreadPoolExecutor(max_workers=max(1, min(16, os.cpu_count() or 1))) as ex:
        objs = list(ex.map(lambda j: _compile(j[0], verbose, j[1], j[2]), jobs))
    tmp = LIB_PATH + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stderr}")
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose="--verbose" in sys.argv))
