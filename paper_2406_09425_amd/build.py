"""Builds libsgprs.so (HIP kernels + C ABI) for gfx950 with hipcc, and the call extension, in-tree."""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libsgprs.so")
CALLS = os.path.join(PKG, "_calls.so")  # CPython extension around the entry points called once per kernel
OBJ_DIR = os.path.join(PKG, "_build")

SOURCES = ["pool.cpp", "pack.cpp", "ops.cpp", "task.cpp", "sched.cpp", "conv_igemm.hip", "conv_ksplit.hip", "conv_wtile.hip", "conv_kpatch.hip", "conv_split.hip", "conv_s2tile.hip", "conv_stem.hip", "conv3x3_patch.hip", "conv3x3_rows.hip", "stem_pool.hip", "stem_f32.hip",
           "pointwise.hip", "fc_gemm.hip", "mfma_probe.hip", "load_probe.hip"]

COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-variable", "-I", os.path.join(ROOT, "include"),
          "-I", CSRC]
# gfx950 only; packed-fp32 instruction selection is switched off on purpose
DEVICE = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [hipcc()] + COMMON + (DEVICE if src.endswith(".hip") else []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build_library(verbose: bool = False) -> str:
    """Compiles every source and links libsgprs.so and _calls.so; always rebuilds."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I", os.path.join(ROOT, "include"),
           "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "pycalls.cpp"), "-o", CALLS, "-L", PKG, "-lsgprs",
           "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"building the call extension failed:\n{r.stdout}\n{r.stderr}")
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True)
