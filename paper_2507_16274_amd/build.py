"""Builds libstalloc.so (hand-written HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libstalloc.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = False, lib: str = LIB, extra=(), only=None) -> str:
    """Compiles the library, or (tests) one of the sources `only` with the definitions `extra`."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = lib + f".tmp{os.getpid()}"
    extra = list(extra) + os.environ.get("STALLOC_DEFINES", "").split()      # e.g. "-DSTALLOC_THREADS_LDS=512"
    cmd = [hipcc] + HIPCC_FLAGS + extra + [s for s in sources() if only is None or os.path.basename(s) in only] + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    noise = "is not a recognized feature for this target"
    out = "\n".join(l for l in res.stdout.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed:\n{out}")
    if verbose and out.strip():
        print(out)
    os.replace(tmp, lib)
    return lib


def build_full_buckets(verbose: bool = False) -> str:
    """For tests: stalloc_make_orders with buckets meant for nearly as many numbers as they have room for, so that
    the way around a full bucket (13 standard deviations off in the library proper) is taken all the time."""
    return build(verbose, os.path.join(os.path.dirname(HERE), "tests", "libfullbuckets.so"), ["-DSTALLOC_OR_BUCKET_MEAN=2040"],
                 ("orders.hip", "layers.hip", "trace_check.hip"))


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
