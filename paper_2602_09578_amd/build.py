"""Builds libmarl_decode.so for gfx950 with hipcc, in-tree (paper_2602_09578_amd/lib/)."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
CSRC = os.path.join(_PKG, "csrc")
LIB_DIR = os.path.join(_PKG, "lib")
LIB_PATH = os.path.join(LIB_DIR, "libmarl_decode.so")
FAST_PATH = os.path.join(LIB_DIR, "fast_calls.so")   # the binding's host code (a Python module)
SOURCES = ["api.hip", "plan_kernel.hip", "attn_kernels.hip", "attn_small_kernel.hip", "logprob_kernels.hip",
           "kv_cache_kernels.hip", "sample_kernels.hip", "grpo_kernels.hip", "prefill_kernels.hip", "balancer.hip", "pack_kernels.hip", "page_pool.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(_ROOT, "include"), "-I" + CSRC]
# Device code of these files never produces or consumes a NaN in floating-point arithmetic
# (masked scores are -inf, unused value slots are cleared as integers), so the compiler may drop
# the canonicalising v_max it otherwise puts in front of every maximum of a matrix-core result:
# the vector ALU is the busiest unit of the attention kernels.  Host code keeps its NaN checks.
_NO_NANS = ["-Xarch_device", "-fno-honor-nans"]
FILE_FLAGS = {"prefill_kernels.hip": _NO_NANS, "attn_kernels.hip": _NO_NANS, "attn_small_kernel.hip": _NO_NANS}


def build_library(verbose: bool = False, extra_flags=(), out_path: str = LIB_PATH) -> str:
    """Compiles every source (always, also when a built library exists) and links."""
    os.makedirs(LIB_DIR, exist_ok=True)
    objdir = os.path.join(LIB_DIR, "_build", os.path.basename(out_path))
    os.makedirs(objdir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(src, []), *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in r.stdout.splitlines() if "not a recognized feature" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{out}")
        if verbose and out.strip():
            print(out)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out_path, *objs]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    return out_path


def fast_calls_sources():
    """What the binding's host code is built from: a module of other sources may call the library with other arguments.  None
    where the sources are not there (the built package alone)."""
    h = hashlib.sha256()
    for path in (os.path.join(CSRC, "fast_calls.cpp"), os.path.join(_ROOT, "include", "marl_decode.h")):
        if not os.path.exists(path):
            return None
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def build_fast_calls(out_path: str = FAST_PATH) -> str:
    """Compiles the binding's host code against torch's headers (always)."""
    import sysconfig
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    os.makedirs(LIB_DIR, exist_ok=True)
    part = f"{out_path}.{os.getpid()}"   # (another process may be loading it, or building it too)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DMARL_FAST_CALLS_SOURCES="{fast_calls_sources()}"',
           "-I" + os.path.join(_ROOT, "include"), "-I" + sysconfig.get_paths()["include"], *["-I" + p for p in include_paths()],
           os.path.join(CSRC, "fast_calls.cpp"), "-o", part, *["-L" + p for p in library_paths()],
           "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for fast_calls.cpp:\n" + r.stdout)
    os.replace(part, out_path)
    return out_path


if __name__ == "__main__":
    print(build_library(verbose=True, extra_flags=sys.argv[1:]))
    print(build_fast_calls())
