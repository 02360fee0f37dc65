"""Build librtt.so (HIP for gfx950) in-tree: one object per source, then link.

Usage: python -m paper_2609_05528_amd.build_lib  (or build() from Python).
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import hashlib
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "librtt.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

# packed FP32 instructions are disabled: they are generated from plain float code otherwise
FLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(HERE, "..", "include")]


# the host FP64 kernels of the small SVD run on AVX2 + FMA (every EPYC has them); contraction stays
# off, so every product and sum is rounded as in the plain build
HOST_SIMD = {"smallla.cpp": ["-Xarch_host", "-march=x86-64-v3", "-Xarch_host", "-ffp-contract=off"]}


# what decides the time of A and A^T and of their variants: the kernels, their records and the lists that
# geometry_load builds for them
OPERATOR_SOURCES = ("operator.hip", "adjoint_cells.hip", "rtt_internal.h", "tables.cpp")


def operator_digest(csrc: str = CSRC) -> str:
    """Digest of the operator's sources: timings and tuner choices taken with others are stale."""
    h = hashlib.sha256()
    for name in OPERATOR_SOURCES:
        with open(os.path.join(csrc, name), "rb") as f:
            h.update(b"%s %d\n" % (name.encode(), os.fstat(f.fileno()).st_size))
            h.update(f.read())
    return h.hexdigest()[:16]


def tune_cache_header(csrc: str = CSRC) -> str:
    """First line of a tuner cache made with these sources (the kernel file's own digest, then the digest of all)."""
    with open(os.path.join(csrc, "operator.hip"), "rb") as f:
        own = hashlib.sha256(f.read()).hexdigest()[:16]
    return "# operator %s sources %s\n" % (own, operator_digest(csrc))


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
    if src.endswith(".cpp"):
        cmd = [HIPCC] + FLAGS + HOST_SIMD.get(os.path.basename(src), []) + ["-x", "hip", "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), r.stderr))
    return obj


def build(verbose: bool = False) -> str:
    """Compile every source and link librtt.so; always rebuilds."""
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed: %s\n%s" % (" ".join(cmd), r.stderr))
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
