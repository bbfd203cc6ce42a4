"""Build libgm.so (the HIP kernels and the C ABI runtime) for gfx950.

Usage: ``python -m paper_2509_16248_amd.build`` or ``build()``.  Objects go
to ``_build/`` at the repository root; the library is written next to this
file, where the Python binding loads it from.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJ = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libgm.so")
ARCH = os.environ.get("GM_OFFLOAD_ARCH", "gfx950")

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
COMMON = ["-O3", "-fPIC", "-std=c++17", f"--offload-arch={ARCH}",
          "-I", INCLUDE, "-I", CSRC,
          # packed fp32 instructions stay off (see the design notes)
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wno-unused-command-line-argument"]

# (source, defines): gm_gemm_16bit.hip holds large kernels and is compiled in
# parts (storage type x group of tile shapes)
SOURCES = ([("gm_gemm_16bit.hip", {"GM_T": t, "GM_GROUP": g}) for t in (0, 1) for g in range(4)]
           + [(s, {}) for s in ("gm_rows.hip", "gm_gemm.hip", "gm_gemm_f32.hip",
                                "gm_gemm_skinny.hip", "gm_attention.hip", "gm_decode.hip",
                                "gm_runtime.cpp")])


def _compile(unit) -> str:
    src, defines = unit
    tag = "".join(f".{v}" for v in defines.values())
    obj = os.path.join(OBJ, os.path.basename(src) + tag + ".o")
    lang = ["-x", "hip"] if src.endswith(".cpp") else []
    cmd = [HIPCC, *COMMON, *[f"-D{k}={v}" for k, v in defines.items()], *lang, "-c",
           os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    """Compile every source and link libgm.so; returns the library path."""
    os.makedirs(OBJ, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
