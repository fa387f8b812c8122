"""Build libvie.so (HIP, gfx950) in place.

``python -m paper_2501_13512_amd.build`` compiles every source under
``csrc/`` with hipcc and links ``paper_2501_13512_amd/libvie.so``.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OUT = os.path.join(PKG, "libvie.so")
OBJ = os.path.join(ROOT, "_build")

# Object of libvie -> its sources.  The product's kernels are compiled in
# several translation units side by side and merged into one object.
OBJECTS = {"mvm": ["mvm.hip", "zconv32.hip", "zconv64.hip"], "krylov": ["krylov.hip"],
           "block_solver": ["block_solver.hip"], "fields": ["fields.hip"], "gmres": ["gmres.hip"],
           "vie_api": ["vie_api.cpp"]}

# Packed FP32 instructions are disabled for every HIP translation unit.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I" + os.path.join(ROOT, "include"),
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    return "hipcc"


def _run(cmd, what: str, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{r.stdout}\n{r.stderr}")


def build(verbose: bool = False) -> str:
    parts = {}   # source -> object file
    for name, srcs in OBJECTS.items():
        d = OBJ if len(srcs) == 1 else os.path.join(OBJ, name)
        os.makedirs(d, exist_ok=True)
        parts.update({s: os.path.join(d, os.path.splitext(s)[0] + ".o") for s in srcs})
    with cf.ThreadPoolExecutor(max_workers=min(len(parts), os.cpu_count() or 1)) as ex:
        list(ex.map(lambda s: _run([_hipcc(), *FLAGS, "-x", "hip", "-c", os.path.join(CSRC, s), "-o", parts[s]],
                                   f"hipcc for {s}", verbose), parts))
    objs = [os.path.join(OBJ, name + ".o") for name in OBJECTS]
    for (name, srcs), obj in zip(OBJECTS.items(), objs):
        if len(srcs) > 1:
            _run(["ld", "-r", *[parts[s] for s in srcs], "-o", obj], f"merging {name}", verbose)
    tmp = OUT + ".tmp"
    _run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp], "link", verbose)
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
