"""Build libqk.so (HIP, gfx950 only) in-tree with hipcc.

Every source compiles to an object with -O3 --offload-arch=gfx950; packed FP32
instructions are disabled (-Xclang -target-feature -Xclang -packed-fp32-ops).
The objects link into ``paper_1908_07187_amd/lib/libqk.so``.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
OBJDIR = os.path.join(HERE, "_build")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(LIBDIR, "libqk.so")

SOURCES = ["api.hip", "kernels.hip", "fused.hip", "fusion.cpp", "stages.cpp", "batch.hip", "sample.hip", "sparse.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE, "-I", CSRC,
    "-Wall", "-Wno-unused-function", "-Wno-unused-result",
]

# Per-source flags.  batch.hip: the pass interpreter keeps a group's sixteen
# amplitudes in registers; plain gates run in an assembly loop, but masked gates,
# phases and measurements are compiled, behind branches that are all uniform.
# Turned into structured control flow, their results are merged with the
# untouched amplitudes at each join; skipping uniform regions leaves real branches
# and in-place updates.  The promotion of register arrays to vector tuples, which
# copies whole tuples likewise, is off too.  With neither flag k_stage spills
# 1600 registers (complex128), without the first 8, without the second 76; with
# both none.
EXTRA = {"batch.hip": ["-mllvm", "-disable-promote-alloca-to-vector",
                       "-mllvm", "-structurizecfg-skip-uniform-regions=true"]}


def _compile(src: str, verbose: bool) -> str:
    path = os.path.join(CSRC, src)
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), *lang, "-c", path, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = [ln for ln in (r.stdout + r.stderr).splitlines()
             if "packed-fp32-ops" not in ln and "warnings generated" not in ln]
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n" + "\n".join(noise))
    if verbose and noise:
        print("\n".join(noise), flush=True)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(LIBDIR, exist_ok=True)
    os.makedirs(OBJDIR, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    jobs = min(len(srcs), int(os.environ.get("MAX_JOBS", "8")))
    with ThreadPoolExecutor(max_workers=max(1, jobs)) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
