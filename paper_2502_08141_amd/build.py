"""Build the HIP library (csrc/*.hip -> liblowra_hip.so) for gfx950 with hipcc, and the binding's native calls
(csrc/call.cpp -> _lowra_call.so) with g++."""
from __future__ import annotations

import glob
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblowra_hip.so")
CALL = os.path.join(HERE, "_lowra_call.so")
OBJ = os.path.join(HERE, "_build")

HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                       # quantize/dequantize arithmetic must stay unfused
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-attributes",
]


# The rank-r products' kernels are loops of about a hundred instructions around a barrier: one that starts in the middle of a
# fetch line costs up to 6 % of a call, and which one does changes with any edit of the file (13824 x 5120, 1500 tokens, s dY B:
# 20.9 to 22.4 us for the same loop at three places, 20.1 aligned).
FILE_FLAGS = {"lora_side.hip": ["-falign-loops=64"]}


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    cmd = ["hipcc", *HIPCC_FLAGS, *FILE_FLAGS.get(os.path.basename(src), ()), "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True, stdout=subprocess.DEVNULL if not verbose else None,
                   stderr=subprocess.PIPE if not verbose else None)
    return obj


def call_command(src: str, out: str) -> list[str]:
    """How csrc/call.cpp becomes an extension module."""
    import sysconfig

    import torch

    t = os.path.dirname(torch.__file__)
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", "-I/opt/rocm/include", f"-I{t}/include",
            f"-I{t}/include/torch/csrc/api/include", "-I" + sysconfig.get_paths()["include"], src,
            "-o", out, f"-L{t}/lib", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", f"-Wl,-rpath,{t}/lib"]


def _compile_call(verbose: bool) -> None:
    cmd = call_command(os.path.join(CSRC, "call.cpp"), CALL)
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True, stderr=None if verbose else subprocess.PIPE)


def build(verbose: bool = False, jobs: int | None = None) -> str:
    """Compile every csrc/*.hip (one hipcc process per file, a few at a time) and link the library."""
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    jobs = jobs or min(8, os.cpu_count() or 1, len(srcs))
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        call = pool.submit(_compile_call, verbose)
        objs = list(pool.map(lambda s: _compile(s, verbose), srcs))
        call.result()
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
