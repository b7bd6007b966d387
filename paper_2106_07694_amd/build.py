"""Build liblbw.so (the HIP kernels and the C ABI) for gfx950, in-tree.

Each source compiles to an object with hipcc, then one shared library is
linked next to this file.  Packed-FP32 instructions are disabled for every
device compile (they are generated from ordinary float code otherwise).
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "liblbw.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

# (source, object name, preprocessor definitions); the tiled transport builds one unit per
# element type, dimension and settling form, the fused one per element type, all in parallel
TILED = [("transport_tiled_unit.hip", f"transport_tiled_{d}d_{t}{'_vs' if v else ''}",
          [f"-DLBW_T={t}", f"-DLBW_D={d}", f"-DLBW_VSS={v}"])
         for t in ("double", "float") for d in (3, 2) for v in (0, 1)]
FUSED = [("transport_fused.hip", f"transport_fused_{t}", [f"-DLBW_T={t}"]) for t in ("double", "float")]
SOURCES = TILED + FUSED + [(src, os.path.splitext(src)[0], []) for src in (
    "adjoint.hip", "lbm.hip", "transport.hip", "transport_tiled.hip", "reduce.hip", "api.cpp")]

COMMON = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wall", "-Wno-unused-function", "-I", os.path.join(HERE, "..", "include")]


def _compile(unit: tuple) -> str:
    src, name, defs = unit
    out = os.path.join(OBJ, name + ".o")
    cmd = [HIPCC, *COMMON, *defs, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src} ({name}):\n{r.stderr}")
    return out


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
