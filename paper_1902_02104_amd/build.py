"""Build libata.so (HIP, gfx950) in-tree.

hipcc compiles every source for gfx950 only; packed FP32 instructions are
disabled for the device code.
"""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libata.so")

SOURCES = ["ata_plan.cpp", "ata_api.cpp", "ata_serve.cpp", "ata_solve.cpp", "ata_scratch.cpp",
           "ata_kernels.hip", "ata_fine.hip", "ata_lp.hip", "ata_chol.hip", "ata_trsv.hip", "ata_mv.hip"]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def build(verbose: bool = False) -> str:
    build_dir = os.path.join(PKG, "_build")
    os.makedirs(build_dir, exist_ok=True)
    objs = []
    common = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "include"),
              "-Wall", "-Wno-unused-function", "-Wno-unused-variable"]
    dev = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
    for src in SOURCES:
        obj = os.path.join(build_dir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc()] + common + dev + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        errs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                         if "packed-fp32-ops" not in l and "unknown target feature" not in l.lower())
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (src, errs))
        if verbose and errs.strip():
            print(errs)
        objs.append(obj)
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs + ["-lpthread"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
