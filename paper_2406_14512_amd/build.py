"""Build of the HIP library libffpic.so (gfx950), in-tree.

Every source is compiled with hipcc for gfx950 only.  The FP64 field and
push kernels are compiled without FP contraction so the FP64 path rounds
each operation as written.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libffpic.so")
ARCH = "gfx950"

SOURCES = [
    ("runtime.cpp", []),
    ("batch.cpp", []),
    ("k_fields64.hip", ["-ffp-contract=off"]),
    # FP32 field step: products fused only within one expression, so that a
    # node computed by two slabs (its halo copy and its own) rounds the same
    # in every unrolled copy of the row step
    ("k_fields32.hip", ["-ffp-contract=on"]),
    ("k_push64.hip", ["-ffp-contract=off"]),
    # LDS adds of the row sums share one address per wave: keep them plain
    # atomics instead of the compiler's lane-by-lane pre-reduction loop
    ("k_push32.hip", ["-mllvm", "-amdgpu-atomic-optimizer-strategy=None"]),
    ("k_sort.hip", []),
    ("k_sort_bucket.hip", []),
    # injected positions follow the oracle's FP64 operation order
    ("k_inject.hip", ["-ffp-contract=off"]),
    # the parent test is evaluated twice and must round the same both times
    ("k_pairs.hip", ["-ffp-contract=off"]),
    ("k_misc.hip", []),
    # spectra follow the oracle's FP64 operation order
    ("k_diag.hip", ["-ffp-contract=off"]),
    ("noalloc.hip", []),
]

COMMON = ["-x", "hip", f"--offload-arch={ARCH}", "-O3", "-fPIC", "-std=c++17",
          "-munsafe-fp-atomics", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wno-unused-result", "-I", os.path.join(ROOT, "include")]


def hipcc() -> str:
    for c in ("/opt/rocm/bin/hipcc", shutil.which("hipcc") or ""):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def _compile(src: str, extra) -> str:
    obj = os.path.join(BUILD, src + ".o")
    cmd = [hipcc(), *COMMON, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile of {src} failed:\n{r.stderr[-6000:]}")
    return obj


def build(jobs: int = 8) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda a: _compile(*a), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-6000:]}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
