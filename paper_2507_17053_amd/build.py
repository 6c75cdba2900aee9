"""Build the HIP library libsbm.so for gfx950 in-tree (hipcc, no JIT cache).

Every source under csrc/ is compiled to an object in _build/ (in parallel), then linked
into paper_2507_17053_amd/libsbm.so.  Flags:
  --offload-arch=gfx950                 CDNA4 code objects only
  -munsafe-fp-atomics                   hardware FP32/FP64 global atomic adds
  -Xclang -target-feature -Xclang -packed-fp32-ops
                                        no packed FP32 instructions in generated code
"""

from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsbm.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["setup.cpp", "kernels_apply.hip", "kernels_taylor.hip", "vec.hip", "rhs.hip", "solver.hip",
           "apply_noalloc.hip", "setup_gpu.hip", "batch.cpp"]
# per-file flags: the device setup evaluates the level sets with the same floating-point
# operations as the host build (no multiply-add contraction), so both agree bit for bit
EXTRA = {"setup_gpu.hip": ["-ffp-contract=off"], "setup.cpp": ["-ffp-contract=off"]}

COMMON = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-munsafe-fp-atomics",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wno-unused-command-line-argument", "-I" + os.path.join(HERE, "..", "include")]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj] + COMMON + EXTRA.get(src, [])
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = min(len(SOURCES), max(1, (os.cpu_count() or 2)))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
