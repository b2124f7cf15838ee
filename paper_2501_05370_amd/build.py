"""Build the HIP library in-tree: ``python -m paper_2501_05370_amd.build``.

hipcc cross-compiles for gfx950 without a GPU.  The shared library lands next to this file and
is what the ctypes binding loads.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsd_mi355x.so")
OBJDIR = os.path.join(HERE, "_build")

FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option"]

# The loops of these kernels run for a whole chain, and the compiler moves the constants of every logarithm and exponential
# in them, rare branches included, to registers ahead of the loop: up to a hundred of them, which cost wavefronts or go to
# scratch memory.
FILE_FLAGS = {"sd_langevin.hip": ["-mllvm", "-disable-machine-licm"]}


def _compile(src: str) -> str:
    name = os.path.basename(src)
    obj = os.path.join(OBJDIR, name + ".o")
    cmd = ["hipcc", *FLAGS, *FILE_FLAGS.get(name, []), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    noise = "packed-fp32-ops"
    warn = "\n".join(l for l in r.stderr.splitlines() if noise not in l and l.strip())
    if warn:
        sys.stderr.write(warn + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    if verbose:
        print(f"[build] hipcc {len(srcs)} sources -> {LIB}", flush=True)
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    return LIB


if __name__ == "__main__":
    build()
