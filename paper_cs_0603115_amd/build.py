"""Build ``libff.so`` (the HIP library behind ``include/ff.h``) for gfx950.

Every HIP source under ``csrc/`` is compiled with hipcc, in parallel, into
``_build/`` and linked in place next to this file, so that the library
travels with the source tree.  No GPU is needed: hipcc cross-compiles.

    python paper_cs_0603115_amd/build.py

(Run it as a file: importing the package loads the library being built.)
"""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libff.so")

ARCH = "gfx950"

# Numerics-defining flags: no contraction (each written operation is one
# rounded instruction; TwoProd's FMA is an explicit builtin), no fast-math,
# binary32 denormals preserved, correctly rounded binary32 division.
# Packed-FP32 instructions are disabled: the compiler would otherwise pair
# independent binary32 operations into v_pk_* forms.
NUMERIC_FLAGS = [
    "-ffp-contract=off",
    "-fno-fast-math",
    "-fno-gpu-flush-denormals-to-zero",
    "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    "-Wno-unused-command-line-argument",
    "-I", INCLUDE,
    "-I", CSRC,
] + NUMERIC_FLAGS

# Further flags of single sources.  ff_gemm.hip: a loop-carried vector of 16
# accumulators stays one value; broken into elements (the default) the 256
# accumulators of the large BF16 tile no longer stay in their registers and
# spill in the loop.
SOURCE_FLAGS = {
    "ff_gemm.hip": ["-mllvm", "-amdgpu-codegenprepare-break-large-phis=false"],
}


def hipcc() -> str:
    path = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(path):
        raise RuntimeError("hipcc not found: the ROCm toolchain is required to build libff")
    return path


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    cmd = [hipcc(), *HIPCC_FLAGS, *SOURCE_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{proc.stdout}\n{proc.stderr}")
    return obj


def build(jobs: int | None = None, verbose: bool = False) -> str:
    """Compile all sources and link ``libff.so``; returns its path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = sources()
    jobs = jobs or min(8, max(1, os.cpu_count() or 1))
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        objs = list(pool.map(_compile, srcs))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError(f"link failed:\n{proc.stdout}\n{proc.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB} from {len(srcs)} sources")
    return LIB


def device_asm(src: str, out: str) -> str:
    """gfx950 assembly of one source (for the instruction audit)."""
    cmd = [hipcc(), *HIPCC_FLAGS, *SOURCE_FLAGS.get(os.path.basename(src), []),
           "--cuda-device-only", "-S", src, "-o", out]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError(f"hipcc -S failed for {src}:\n{proc.stderr}")
    return out


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
