"""Builds libpicasso_hip.so in-tree with hipcc for gfx950, and the Python module that calls it (_host) with g++."""
from __future__ import annotations

import os
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpicasso_hip.so")
SOURCES = [os.path.join(CSRC, "picasso.hip")]
HOST = os.path.join(HERE, "_host" + sysconfig.get_config_var("EXT_SUFFIX"))

# -ffp-contract=off: every fp32 operation is rounded on its own, in the order written (bit-exact results).
# packed-fp32 instructions are disabled on purpose.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: the HIP library cannot be built")
    return exe


def build_library(verbose: bool = False) -> str:
    cmd = [hipcc()] + FLAGS + ["-I", os.path.join(os.path.dirname(HERE), "include"), "-o", LIB] + SOURCES
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    build_host(verbose)
    return LIB


def build_host(verbose: bool = False) -> str:
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", sysconfig.get_path("include")]
    for d in include_paths():
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, "host.cpp"), "-o", HOST, "-L", HERE, "-l:" + os.path.basename(LIB),
            "-Wl,-rpath,$ORIGIN"]
    for d in library_paths():
        cmd += ["-L", d]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10"]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return HOST


if __name__ == "__main__":
    print(build_library(verbose=True))
