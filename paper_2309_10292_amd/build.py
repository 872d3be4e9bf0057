"""Builds libgs.so (HIP for gfx950) in-tree with hipcc.

Every HIP source is compiled with:
  --offload-arch=gfx950            MI355X only
  -ffp-contract=off                no implicit FMA: the FP64 step must follow the
                                   FP64 operation order exactly; fused operations
                                   are written out explicitly where intended
  -Xclang -target-feature -Xclang -packed-fp32-ops
                                   no packed-FP32 instructions
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIBDIR, "libgs.so")
BUILD = os.path.join(ROOT, "_build")

# (a source given as (file, n) is compiled with GS_TB_STORAGE=n: the blocked
# kernels of one storage type each)
SOURCES = [*(("gs_tblock.hip", n) for n in range(5)), "gs_step.hip", "gs_block.hip", "gs_aux.hip", "gs_surrogate.hip",
           "gs_api.cpp", "gs_batch.cpp", "gs_surrogate_api.cpp", "gs_tunecache.cpp", "gs_hostio.cpp",
           "gs_noalloc.hip"]

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-Wall", "-Wno-unused-function"]


def hipcc() -> str:
    p = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(p):
        raise RuntimeError("hipcc not found: the HIP library cannot be built")
    return p


def _object(src) -> str:
    return os.path.join(BUILD, src + ".o" if isinstance(src, str) else f"{src[0]}.{src[1]}.o")


def _compile(src, extra: list[str]) -> str:
    os.makedirs(BUILD, exist_ok=True)
    obj = _object(src)
    if not isinstance(src, str):
        src, extra = src[0], [*extra, f"-DGS_TB_STORAGE={src[1]}"]
    cmd = [hipcc(), *FLAGS, *extra, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    return obj


def build(extra: list[str] | None = None, jobs: int = 8) -> str:
    """Compile every HIP source and link libgs.so; always rebuilds."""
    extra = list(extra or [])
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, extra), SOURCES))
    os.makedirs(LIBDIR, exist_ok=True)
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link of libgs.so failed")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
