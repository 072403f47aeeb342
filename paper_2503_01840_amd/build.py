"""Builds libeagle3.so (HIP, gfx950) in-tree with plain hipcc."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libeagle3.so")
SOURCES = ["eagle3_api.hip", "gemm_skinny.hip", "gemm_wide.hip", "gemm_f32.hip", "elementwise.hip", "attention.hip", "select.hip",
           "accept.hip", "commit.hip", "causal_attention.hip"]
# Kernel arguments, as far as they fit (14 registers), are in registers when a wavefront starts instead of behind its first memory round trip.  That is for
# arguments of their own, not for members of a struct: what a kernel needs for its first loads comes first in its list.
FLAGS = ["-O3", "-mllvm", "-amdgpu-kernarg-preload-count=16", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def _compile(src):
    obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    return obj, err


def build_library(verbose=False):
    """Compiles every source and links the shared library; always rebuilds."""
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        results = list(ex.map(_compile, SOURCES))
    if verbose:
        for _, err in results:
            if err.strip():
                print(err, file=sys.stderr)
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *[o for o, _ in results]]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
