"""Build libconvrot.so and the extension module _torch_calls.so in-tree with hipcc for gfx950.  Run as ``python -m paper_2512_03673_amd.build``."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from typing import Optional

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libconvrot.so")
CALLS = os.path.join(HERE, "_torch_calls.so")
SOURCES = ("convrot_api.hip", "rotquant.hip", "lanes8.hip", "gemm_w4a4.hip", "gemm_w8a8.hip", "forward_small.hip")
OWN_FLAGS = {"lanes8.hip": ("-fno-slp-vectorize",)}      # the file says why

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # packed-fp32 instructions stay off on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # kernels find their first arguments in registers when they start, instead of waiting 0.3-0.6 us for a scalar load from a cold cache
    # (us: M1 x N9216 x K3072 forward 6.44 -> 6.14, M77 x N3072 x K3072 at 8 bits 10.87 -> 10.65, rotate+quantise [4608, 3072] at g = 256 10.4 -> 9.9)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def build(verbose: bool = True, extra_flags=(), out: str = LIB) -> str:
    """Compile every HIP source (always recompiles) and link the shared library."""
    if verbose:   # the kernels lean on this compiler's code generation: show which one built them
        print(subprocess.run(["hipcc", "--version"], capture_output=True, text=True).stdout.strip(), flush=True)
    objdir = os.path.join(HERE, "_build", os.path.basename(out).replace(".so", ""))
    os.makedirs(objdir, exist_ok=True)

    def compile_one(src: str) -> str:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = ["hipcc", *FLAGS, *OWN_FLAGS.get(src, ()), *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = out + f".tmp{os.getpid()}"
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    if out == LIB:
        build_calls(verbose)
    return out


def build_calls(verbose: bool = True, out: str = CALLS) -> Optional[str]:
    """Compile the extension module (host code only; it calls the C ABI of the library that binding.py loads).  Returns None
    where there is no torch to build it for: the library stands without it, for programs that call the C ABI."""
    try:
        import torch    # headers and libraries; neither torch nor a GPU is used
        root = os.path.dirname(torch.__file__)
    except ImportError:
        root = None
    if root is None or not os.path.isdir(os.path.join(root, "include", "torch", "csrc")):
        print(f"no torch with headers: {os.path.basename(out)}, which binding.py needs, is not built", file=sys.stderr, flush=True)
        return None
    lib = os.path.join(root, "lib")
    tmp = out + f".tmp{os.getpid()}"
    cmd = ["hipcc", "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-DUSE_ROCM",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", os.path.join(ROOT, "include"),
           "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_path("include"), "-o", tmp, os.path.join(CSRC, "torch_calls.cpp"), "-L", lib, "-ltorch_python",
           "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    # usage: python -m paper_2512_03673_amd.build [--out path.so] [extra hipcc flags ...]
    argv = sys.argv[1:]
    target = LIB
    if argv[:1] == ["--out"]:
        target, argv = os.path.abspath(argv[1]), argv[2:]
    print(build(extra_flags=argv, out=target))
