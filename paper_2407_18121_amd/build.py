"""Build libelastic_cache.so in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libelastic_cache.so")
FAST = os.path.join(HERE, "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["ec_api.hip", "decode.hip", "merge.hip", "select.hip", "score_simt.hip", "score_mfma.hip",
           "score_f32.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fno-gpu-rdc",
    "-Wall", "-Wno-unused-function",
    # packed fp32 instruction selection is switched off on this hardware
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build(verbose: bool = False) -> str:
    cmd = [HIPCC] + FLAGS + ["-o", LIB] + [os.path.join(CSRC, s) for s in SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    build_fastcall(verbose)
    return LIB


def build_fastcall(verbose: bool = False) -> str:
    """The binding's native half: a CPython module over torch's headers, host code only."""
    import torch
    from torch.utils import cpp_extension
    lib_dirs = cpp_extension.library_paths()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", f'-DEC_TORCH_VERSION="{torch.__version__}"', "-o", FAST, os.path.join(CSRC, "fastcall.cpp")]
    cmd += [f"-I{d}" for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]]
    cmd += [f"-L{d}" for d in lib_dirs] + ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return FAST


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
