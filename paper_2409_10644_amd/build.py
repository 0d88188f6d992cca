"""Builds libmcsd.so (HIP, gfx950) and _pycall.so (host) in-tree.  Run as `python -m paper_2409_10644_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmcsd.so")
PYCALL = os.path.join(HERE, "_pycall.so")           # CPython marshalling of the hot entry points (host code only)
OBJ = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          # leading scalar kernel arguments arrive in registers, so a kernel's first loads need not wait for the argument block
          "-mllvm", "-amdgpu-kernarg-preload-count=16", "-Wall", "-Wno-unused-function"]
# per-file extra flags: the verification kernels must perform exactly the IEEE operations written
SOURCES = {
    "mask.cpp": ["-x", "hip"],
    # matrix instructions on ordinary registers also in kernels whose LDS leaves one workgroup per compute unit (the compiler
    # otherwise keeps their accumulators in the other half of the register file and copies them to and fro)
    "tree_attention.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
    "verify_tree.hip": ["-ffp-contract=off"],
    "commit_path.hip": [],
    "decision.hip": [],
    "probe.hip": [],
}


def build_library(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    objs = []
    procs = []
    for src, extra in SOURCES.items():
        obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
        cmd = [HIPCC, *COMMON, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, pr in procs:
        out, _ = pr.communicate()
        if pr.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I", os.path.join(ROOT, "include"),
           "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "pycall.cpp"), "-o", PYCALL]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
