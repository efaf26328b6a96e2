"""Builds the C-ABI library `libmgrit.so` for gfx950 with hipcc (in-tree, next to this file)."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libmgrit.so")
SOURCES = ["mgrit_api.hip", "mgrit_kernels.hip", "mgrit_conv_grad.hip", "mgrit_sweep.hip", "mgrit_wave.hip", "mgrit_wide.hip"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def build(verbose: bool = True) -> str:
    """Compile every HIP source into libmgrit.so (always recompiles)."""
    objs = []
    flags = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             # kernels that keep a few hundred accumulator / state registers per lane have fully unrolled
             # loops past the default cost limit of `#pragma unroll`; a loop left rolled would index those
             # registers dynamically and push them to scratch memory
             "-mllvm", "-pragma-unroll-threshold=200000",
             "-I", os.path.join(ROOT, "include")]
    procs = []
    for src in SOURCES:
        obj = os.path.join(HERE, "csrc", src.replace(".hip", ".o"))
        cmd = [hipcc(), *flags, "-c", os.path.join(HERE, "csrc", src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for cmd, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if pr.returncode != 0:
            raise RuntimeError("hipcc failed: " + " ".join(cmd) + "\n" + out)
        if verbose and out.strip():
            print(out)
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
