"""Build libwos.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2406_01713_amd.build

Every source is compiled for gfx950 only; packed-FP32 instructions are
disabled (-packed-fp32-ops) and none are written by hand.  A declaration
that shadows another (a loop-local variable hiding a parameter of the same
name) is a build error."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libwos.so")
BUILD = os.path.join(ROOT, "_build")
ARCH = os.environ.get("WOS_OFFLOAD_ARCH", "gfx950")

# (source, macro definitions): the walk kernels are compiled once per
# variant, so their long compilations run side by side
SOURCES = [*(("wos_persistent.hip", [f"-DWOS_PERSISTENT_SRC={s}", f"-DWOS_PERSISTENT_LISTS={l}",
                                     f"-DWOS_PERSISTENT_MAXD={m}"])
             for s in (0, 1) for l, m in ((0, 8), (1, 8), (1, 5))),
           *(("wos_plain.hip", [f"-DWOS_PLAIN_T={t}", f"-DWOS_PLAIN_LOW={h}"])
             for t in ("float", "double") for h in (0, 1)),
           ("wos_kernels.hip", []), ("wos_grid.hip", []), ("wos_api.cpp", []), ("wos_microbench.hip", [])]
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-x", "hip",
         *os.environ.get("WOS_EXTRA_FLAGS", "").split(),
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Werror=shadow", "-I", os.path.join(ROOT, "include")]


def _hipcc():
    h = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(h):
        raise RuntimeError("hipcc not found: libwos needs the ROCm toolchain")
    return h


def _compile(unit):
    src, defs = unit
    os.makedirs(BUILD, exist_ok=True)
    obj = os.path.join(BUILD, os.path.basename(src) + "".join(defs).replace("=", "_") + ".o")
    cmd = [_hipcc(), *FLAGS, *defs, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        print(err, file=sys.stderr)
    return obj


def build(verbose=True):
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
