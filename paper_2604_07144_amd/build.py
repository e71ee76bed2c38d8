"""Build the HIP library for gfx950 in-tree (``paper_2604_07144_amd/libautopoiesis_eval.so``), and a library of kernels for the tests."""
from __future__ import annotations

import os
import subprocess

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
SOURCES = [os.path.join(_HERE, "csrc", "ap_eval.hip")]
LIB_PATH = os.path.join(_HERE, "libautopoiesis_eval.so")
TEST_SOURCES = [os.path.join(ROOT, "tests", "device", "runs.hip")]
TEST_LIB_PATH = os.path.join(ROOT, "tests", "device", "libruns.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
    # packed-FP32 instruction forms are kept out of all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


def _compile(verbose: bool, sources: list, lib_path: str, *flags: str) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *flags, *sources, "-o", lib_path]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return lib_path


def build(verbose: bool = False) -> str:
    """Compile every HIP source with hipcc; always recompiles."""
    return _compile(verbose, SOURCES, LIB_PATH)


def build_tests(verbose: bool = False) -> str:
    """Compile the kernels that only tests run, which take the library's device code piece by piece."""
    return _compile(verbose, TEST_SOURCES, TEST_LIB_PATH, "-I", os.path.join(_HERE, "csrc"), "-Wno-unused-function", "-Wno-unneeded-internal-declaration")


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_tests(verbose=True))
