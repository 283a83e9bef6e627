"""Compile libsfi.so (HIP, gfx950 only) and its CPython module _sfi.so in-tree next to this file."""
from __future__ import annotations

import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsfi.so")
PY_LIB = os.path.join(HERE, "_sfi.so")

# packed-fp32 code generation is switched off on purpose for this target
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               # leading scalar kernel arguments arrive in registers
               "-mllvm", "-amdgpu-kernarg-preload-count=14",
               "-Wall", "-Wno-unused-function"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_lib(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, *sources(), "-o", LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err)
    build_py_module()
    return LIB


def build_py_module() -> str:
    """The hot calls as a CPython module (host code only); it gets libsfi's entry points from binding.py, not from the linker."""
    cxx = os.environ.get("CXX", "g++")
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", sysconfig.get_paths()["include"],
           "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "sfi_py.cpp"), "-o", PY_LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cxx} failed:\n" + r.stderr)
    return PY_LIB


if __name__ == "__main__":
    print(build_lib(verbose=True))
