"""Compile the HIP sources of the library for gfx950 into paper_1911_05181_amd/libulsnn.so (in-tree)."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libulsnn.so")
FAST_CALL = os.path.join(HERE, "_fast_call.so")     # argument marshalling of the binding (CPython extension, host only)
SOURCES = ["ulsnn.hip", "gemm_fp32.hip", "gemm_split.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def fast_call_command():
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths

    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
             f'-DBUILT_WITH_TORCH="{torch.__version__}"']
            + [f"-isystem{d}" for d in include_paths()] + ["-I" + sysconfig.get_paths()["include"]]
            + ["-o", FAST_CALL, os.path.join(CSRC, "fast_call.cpp")]
            + [f"-L{d}" for d in library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-lc10"])


def build(verbose: bool = False) -> str:
    """Always compiles (the "does it build" check), the sources side by side; returns the path of the shared library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        objects, running = [], []
        for s in SOURCES:
            objects.append(os.path.join(tmp, s + ".o"))
            cmd = [hipcc] + HIPCC_FLAGS + ["-c", "-o", objects[-1], os.path.join(CSRC, s)]
            if verbose:
                print(" ".join(cmd), flush=True)
            running.append((cmd, subprocess.Popen(cmd, cwd=CSRC)))
        cmd = fast_call_command()
        if verbose:
            print(" ".join(cmd), flush=True)
        running.append((cmd, subprocess.Popen(cmd, cwd=CSRC)))
        failed = [cmd for cmd, p in running if p.wait() != 0]
        if failed:
            raise subprocess.CalledProcessError(1, failed[0])
        subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objects, check=True, cwd=CSRC)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
