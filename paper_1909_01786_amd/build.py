"""Build libasp.so (HIP for gfx950) in-tree with hipcc.

The library is the product path: ``csrc/encode.cpp`` (host encoding),
``csrc/solver.hip`` and ``csrc/solver_wide.hip`` (device search, with Deps of
one word and of several), ``csrc/scorer.hip`` (learned Decision scorer), ``csrc/trainer.hip`` and ``csrc/train.cpp`` (its training) and
``csrc/api.cpp`` (C ABI of ``include/asp.h``).  Packed FP32 instructions are disabled for every HIP
translation unit.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libasp.so")
SOURCES = ["encode.cpp", "api.cpp", "train.cpp", "solver.hip", "solver_wide.hip", "scorer.hip", "trainer.hip"]
HEADERS = ["encode.h", "layout.h", "scorer.h", "train.h", "trainer.h"]
ARCH = os.environ.get("ASP_OFFLOAD_ARCH", "gfx950")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", f"-I{os.path.join(ROOT, 'include')}"]


def build(verbose: bool = False) -> str:
    """Compile every source and link libasp.so (always recompiles)."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    cmds, objs = [], []
    for src in SOURCES:
        obj = os.path.join(objdir, src + ".o")
        lang = ["-x", "hip"]
        cmds.append([HIPCC, *FLAGS, *lang, "-c", os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    # the translation units compile independently, in parallel
    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
    with ThreadPoolExecutor(len(cmds)) as ex:
        list(ex.map(run, cmds))
    tmp = f"{LIB}.tmp{os.getpid()}"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)
