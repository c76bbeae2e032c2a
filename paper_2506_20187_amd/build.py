"""Compile the HIP sources in csrc/ into libleoam.so for gfx950, and csrc/bind.cpp into _bind.so (in-tree).

Every source file becomes an object of its own (compiled in parallel, objects under
_build/), then one link.  `python paper_2506_20187_amd/build.py` recompiles only what
changed since its object was written; build_library() without arguments recompiles
everything.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libleoam.so")
BIND_SRC = os.path.join(CSRC, "bind.cpp")
BIND = os.path.join(HERE, "_bind.so")      # argument marshalling of the per-step entry points

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def headers():
    return glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(HERE, "..", "include", "*.h"))


def needs_build() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(BIND):
        return True
    t = os.path.getmtime(LIB)
    return (any(os.path.getmtime(p) > t for p in sources() + headers())
            or os.path.getmtime(BIND_SRC) > os.path.getmtime(BIND))


def _bind_command():
    import torch
    torch_dir = os.path.dirname(torch.__file__)
    return ([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
             "-isystem", os.path.join(torch_dir, "include"),
             "-isystem", os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"),
             "-isystem", sysconfig.get_paths()["include"], BIND_SRC,
             "-L" + os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", BIND])


def build_library(verbose: bool = True, incremental: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    newest_header = max(os.path.getmtime(p) for p in headers())
    jobs = []
    for src in sources():
        obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
        stale = (not os.path.exists(obj)) or os.path.getmtime(obj) < max(os.path.getmtime(src), newest_header)
        if stale or not incremental:
            jobs.append([hipcc] + HIPCC_FLAGS + ["-c", src, "-o", obj])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    workers = max(1, min(len(jobs), int(os.environ.get("MAX_JOBS", "8")), os.cpu_count() or 1))
    with ThreadPoolExecutor(workers) as pool:
        list(pool.map(run, jobs))
    objs = [os.path.join(OBJ, os.path.basename(s)[:-4] + ".o") for s in sources()]
    run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB])
    if not incremental or not os.path.exists(BIND) or os.path.getmtime(BIND) < max(os.path.getmtime(BIND_SRC), newest_header):
        run(_bind_command())
    return LIB


if __name__ == "__main__":
    build_library(incremental="--all" not in sys.argv)
    sys.exit(0)
