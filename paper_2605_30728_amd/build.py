"""Build libibp.so (the C ABI in include/ibp.h) for gfx950 with hipcc, in-tree.

    python -m paper_2605_30728_amd.build      # or build() from Python

Device code is compiled with packed FP32 instructions disabled (none of the kernels
do floating point, and the flag keeps hipcc from emitting them anywhere).
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libibp.so")
ARCH = os.environ.get("IBP_OFFLOAD_ARCH", "gfx950")

HIP_SOURCES = ["ibp_kernels.hip", "ibp_gather_kernels.hip", "ibp_part_kernels.hip", "ibp_cache_kernels.hip", "ibp_runtime.hip"]
CXX_SOURCES = ["ibp_host.cpp", "ibp_pool.cpp", "ibp_meta_slots.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", f"-I{INCLUDE}", f"-I{CSRC}"]
HIP_FLAGS = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"build step failed: {' '.join(cmd)}")
    noise = [ln for ln in (r.stderr or "").splitlines()
             if ln.strip() and "packed-fp32-ops" not in ln and "hip-link" not in ln]
    if noise and verbose:
        sys.stderr.write("\n".join(noise) + "\n")


def build(verbose=False):
    """Compile every source and link libibp.so. Always rebuilds."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    objs = []
    for src in HIP_SOURCES:
        obj = os.path.join(BUILD_DIR, src + ".o")
        _run([HIPCC, *COMMON, *HIP_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj], verbose)
        objs.append(obj)
    for src in CXX_SOURCES:
        obj = os.path.join(BUILD_DIR, src + ".o")
        _run(["g++", *COMMON, "-c", os.path.join(CSRC, src), "-o", obj], verbose)
        objs.append(obj)
    tmp = LIB + ".tmp"
    _run([HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", tmp, "-lpthread"], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
