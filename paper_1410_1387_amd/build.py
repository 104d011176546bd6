"""Build libfdwave.so for gfx950 in-tree with hipcc.

Each translation unit under csrc/ is compiled separately (in parallel) and linked
into ``paper_1410_1387_amd/libfdwave.so``.  Device code is built without packed
FP32 instructions (``-packed-fp32-ops``) and with FMA contraction left to the
explicit fma calls in the kernels.
"""

from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfdwave.so")
# translation units: a source and, for the forward kernels (one object per radius), a define
SOURCES = [(f"fd_fwd_{t}.hip", f"-DFD_RADIUS={r}") for t in ("f32", "f64") for r in (4, 8, 1, 2, 3, 5, 6, 7)] + [
    (s, "") for s in ("fd_adj_f32.hip", "fd_adj_f64.hip", "fd_vti_f32.hip", "fd_vti_f64.hip", "fd_fwd2_f32.hip",
                      "fd_multi2d_f32.hip", "fd_multi2d_f64.hip", "fd_api.hip", "fd_util.hip", "fd_vti_api.hip")]
ARCH = "gfx950"


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def compile_flags() -> list[str]:
    return [
        f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-Wall", "-Wno-unused-function",
        "-I", os.path.join(HERE, "..", "include"),
    ]


def _compile(unit: tuple[str, str]) -> str:
    src, define = unit
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + define.replace("-DFD_RADIUS=", "_r") + ".o")
    cmd = [_hipcc(), *compile_flags(), *([define] if define else []), "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    return obj


def build(jobs: int | None = None, verbose: bool = False) -> str:
    """Compile every source and link libfdwave.so; always rebuilds."""
    os.makedirs(BUILD, exist_ok=True)
    jobs = jobs or min(len(SOURCES), os.cpu_count() or 4)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
