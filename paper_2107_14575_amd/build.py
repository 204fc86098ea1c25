"""Builds libdq.so (the C-ABI HIP library, hipcc for gfx950) and _dqcall.so (its calls from Python, g++) in-tree."""
from __future__ import annotations

import glob
import os
import subprocess
import sysconfig
import tempfile
import warnings
from concurrent.futures import ThreadPoolExecutor

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
CSRC = os.path.join(_PKG, "csrc")
LIB_PATH = os.path.join(_PKG, "libdq.so")
CALL_PATH = os.path.join(_PKG, "_dqcall.so")

HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared",
    # every float operation that decides a level is a single IEEE rounding: no FMA contraction
    "-ffp-contract=off",
    # packed-FP32 code generation stays off
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_calls(verbose: bool = False) -> str:
    """Compile the CPython module.  It is not linked to libdq.so: binding.py binds it to the one that it opens."""
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", os.path.join(_ROOT, "include"),
           "-I", sysconfig.get_paths()["include"], "-o", CALL_PATH, os.path.join(CSRC, "dq_python.cpp")]
    if verbose:
        print(" ".join(cmd), flush=True)
    if os.path.exists(CALL_PATH):
        os.remove(CALL_PATH)  # never one of an earlier build beside a new library
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n{res.stdout}")
    return CALL_PATH


def build_library(verbose: bool = False) -> str:
    """Compile every HIP source into libdq.so, and the calls from Python; always compiles.  The C library stands by itself: if the
    calls cannot be compiled (they take a C++ compiler and Python's headers), that is a warning, and importing them an error."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    include = ["-I", os.path.join(_ROOT, "include"), "-I", CSRC]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in res.stdout.splitlines()
                        if "packed-fp32-ops" not in l or "error" in l)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + out)
        if verbose and out.strip():
            print(out, flush=True)

    # the sources side by side: one of them holds most of the kernels
    with tempfile.TemporaryDirectory() as objects:
        jobs = [(src, os.path.join(objects, os.path.basename(src) + ".o")) for src in sources()]
        flags = [f for f in HIPCC_FLAGS if f != "-shared"]
        with ThreadPoolExecutor(len(jobs)) as pool:
            list(pool.map(lambda job: run([hipcc, *flags, *include, "-c", job[0], "-o", job[1]]), jobs))
        run([hipcc, *HIPCC_FLAGS, "-o", LIB_PATH, *(obj for _, obj in jobs)])
    try:
        build_calls(verbose)
    except (RuntimeError, OSError) as e:
        warnings.warn(f"no {os.path.basename(CALL_PATH)}, so no calls from Python: {e}", RuntimeWarning, stacklevel=2)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
