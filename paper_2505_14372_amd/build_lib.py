"""Build libpty.so (HIP, gfx950) in-tree with hipcc.

Usage: python -m paper_2505_14372_amd.build_lib [--verbose]
"""
from __future__ import annotations

import hashlib
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libpty.so")
BUILD_DIR = os.path.join(PKG, "_build")   # object files (git-ignored)

SOURCES = ["pty_kernels.hip", "pty_chain.hip", "pty_finish.hip", "pty_api.cpp"]

HIP_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-munsafe-fp-atomics",
    # no packed FP32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

# the register-tile kernels sit at the 128 registers of four waves per SIMD: with
# the target's own pressure tracking the scheduler spills fewer of them
SOURCE_FLAGS = {"pty_chain.hip": ["-mllvm", "-amdgpu-use-amdgpu-trackers=1"]}


def hipcc():
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False, jobs: int = 4, defines=(), out: str = LIB) -> str:
    """Compile every source and link libpty.so (or `out`); returns its path.
    `defines` are extra -D macros (tuning constants of the kernels)."""
    cc = hipcc()
    objs = []
    procs = []
    # a stable tag per (defines, output), so concurrent builds of variants do not collide
    tag = hashlib.sha256(repr((tuple(defines), os.path.abspath(out))).encode()).hexdigest()[:16]
    os.makedirs(BUILD_DIR, exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(BUILD_DIR, f"{src}.{tag}.o")
        cmd = [cc, *HIP_FLAGS, *SOURCE_FLAGS.get(src, []), *[f"-D{d}" for d in defines], "-I", INCLUDE, "-I", CSRC, "-c",
               os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
        if len(procs) >= jobs:
            _wait(procs.pop(0), verbose)
    for p in procs:
        _wait(p, verbose)
    tmp = out + ".tmp"
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs, "-lhipfft"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    os.replace(tmp, out)
    for o in objs:
        os.remove(o)
    return out


def _wait(item, verbose):
    src, p = item
    out, _ = p.communicate()
    if p.returncode != 0:
        raise RuntimeError(f"compiling {src} failed:\n{out}")
    if verbose and out.strip():
        print(out)


if __name__ == "__main__":
    print(build(verbose="--verbose" in sys.argv))
