"""Compile libgpusparse.so for gfx950 with hipcc (in-tree, no JIT cache).

    python paper_2606_26441_amd/build.py

(Run by path: importing the package loads the library, which is what this
script replaces.)
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
BUILD_DIR = os.path.join(ROOT, "_build")
LIB_PATH = os.path.join(HERE, "libgpusparse.so")

SOURCES = ["gs_host.cpp", "gs_server.cpp", "gs_topk.hip", "gs_yardstick.hip", "gs_noalloc.hip"]
# gs_score.hip compiles in parts, in parallel (one weight form each, then the rest): its kernels
# are most of the build's time
UNITS = [("gs_score.hip", "-DGS_SCORE_PART=%d" % part) for part in range(4)] + [(src, None) for src in SOURCES]
HEADERS = [os.path.join(CSRC, "gs_internal.h"), os.path.join(ROOT, "include", "gpusparse.h")]

ARCH = "gfx950"
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-munsafe-fp-atomics",
    # packed fp32 instructions stay disabled on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result", "-Wno-unused-function",
]


def hipcc() -> str:
    for c in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.exists(c) or c == "hipcc":
            return c
    return "hipcc"


def _compile(unit) -> str:
    src, define = unit
    os.makedirs(BUILD_DIR, exist_ok=True)
    obj = os.path.join(BUILD_DIR, src + (define[-1] if define else "") + ".o")
    cmd = [hipcc(), *FLAGS, *([define] if define else []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, " ".join(cmd), r.stderr))
    return obj


def build(verbose: bool = False) -> str:
    """Compile every source and link libgpusparse.so (always rebuilds)."""
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(UNITS)) as ex:
        objs = list(ex.map(_compile, UNITS))
    tmp = LIB_PATH + ".tmp%d" % os.getpid()
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (" ".join(cmd), r.stderr))
    os.replace(tmp, LIB_PATH)
    if verbose:
        print("built", LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
