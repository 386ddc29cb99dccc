"""Build libkvr.so for gfx950 with hipcc (in-tree, under ``_build/``)."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OUT_DIR = os.path.join(PKG, "_build")
LIB = os.path.join(OUT_DIR, "libkvr.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["kvr_api.cpp", "kvr_grid.hip", "kvr_aux.hip", "kvr_sorted.hip", "kvr_binned.hip",
           "kvr_replay.hip",
           "kvr_controller.hip", "kvr_r3.hip",
           "kvr_factored.hip", "kvr_noalloc.hip", "kvr_small.hip"]
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
          # no packed-fp32 instruction selection anywhere
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]
# Device code only: every sample is validated on its bits before use and no
# NaN ever reaches the arithmetic, so min/max need no NaN quieting.
DEVICE = ["-Xarch_device", "-fno-honor-nans"]


def _compile(src: str) -> str:
    obj = os.path.join(OUT_DIR, os.path.basename(src) + ".o")
    cmd = [HIPCC] + COMMON + (DEVICE if src.endswith(".hip") else []) + \
        ["-c", os.path.join(CSRC, src), "-o", obj]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return obj


def build(verbose: bool = False) -> str:
    """Compile every source and link libkvr.so; always rebuilds."""
    os.makedirs(OUT_DIR, exist_ok=True)
    try:
        with cf.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
            objs = list(ex.map(_compile, SOURCES))
        tmp = LIB + f".tmp{os.getpid()}"
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs,
                       check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
        os.replace(tmp, LIB)
    except subprocess.CalledProcessError as err:
        sys.stderr.write(err.stdout.decode(errors="replace"))
        raise
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
