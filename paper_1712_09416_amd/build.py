"""Build libtpcca.so (HIP kernels + C ABI) for gfx950 in the package folder."""
from __future__ import annotations

import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtpcca.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = os.environ.get("TPC_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared",
    f"--offload-arch={ARCH}",
    # every float product and sum rounded as written (decisions must be
    # reproducible on the CPU); IEEE division and square root
    "-ffp-contract=off", "-fno-fast-math", "-fhip-fp32-correctly-rounded-divide-sqrt",
    # no packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"),
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def compile_library(out: str, srcs: list, flags=(), verbose: bool = False) -> str:
    tmp = out + ".tmp"
    cmd = [HIPCC, *FLAGS, *flags, "-o", tmp, *srcs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    return out


def build(verbose: bool = False) -> str:
    return compile_library(LIB, sources(), verbose=verbose)


# kernels that only the tests launch
TEST_SRC = os.path.join(ROOT, "tests", "native", "roots.hip")
TEST_LIB = os.path.join(ROOT, "tests", "native", "libroots.so")


def build_tests(verbose: bool = False) -> str:
    return compile_library(TEST_LIB, [TEST_SRC], flags=("-I", CSRC), verbose=verbose)


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)
