"""Compile the HIP attention library for gfx950 into paper_2410_20399_amd/libtk_attn.so, and its Python binding."""
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtk_attn.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["tk_attn_api.hip", "attn_fwd.hip", "attn_bwd.hip", "mfma_probe.hip", "rotary.hip", "gemm.hip"]
HEADERS = ["tk_common.h", "tk_launch.h", os.path.join("..", "..", "include", "tk_attn.h")]
BINDING_SOURCES = ["binding.cpp", os.path.join("..", "..", "include", "tk_attn.h")]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 instructions are kept off for every HIP translation unit
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-inline-asm",
]
# Kernels with more than 256 registers: the results of matrix instructions go to whichever half of the register file holds
# them longest.  (By default all of them go to the accumulator half, and what the vector ALU reads is copied out of it.)
SOURCE_FLAGS = {name: ["-mllvm", "-amdgpu-mfma-vgpr-form=1"] for name in ("attn_fwd.hip", "attn_bwd.hip")}


def _newer(sources, target) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(os.path.join(CSRC, f)) > t for f in sources)


def stale() -> bool:
    return _newer(SOURCES + HEADERS, LIB) or _newer(BINDING_SOURCES, BINDING)


def _build_library(extra_flags) -> None:
    out = os.path.join(HERE, "build")
    os.makedirs(out, exist_ok=True)

    def compile_one(source):
        obj = os.path.join(out, source + ".o")
        subprocess.run(["hipcc", *FLAGS, *SOURCE_FLAGS.get(source, []), *extra_flags, "-c", os.path.join(CSRC, source), "-o", obj], check=True)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as pool:
        objects = list(pool.map(compile_one, SOURCES))
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objects, "-o", LIB], check=True)


def _build_binding() -> None:
    import torch
    root = os.path.dirname(os.path.abspath(torch.__file__))
    abi = int(torch._C._GLIBCXX_USE_CXX11_ABI)
    subprocess.run(
        ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-w",
         "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={abi}",
         "-I" + os.path.join(root, "include"), "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
         "-I/opt/rocm/include", "-I" + sysconfig.get_paths()["include"],
         os.path.join(CSRC, "binding.cpp"), "-o", BINDING,
         "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"],
        check=True)


def build(force: bool = True, extra_flags=()) -> str:
    if not force and not stale():
        return LIB
    _build_library(extra_flags)
    _build_binding()
    return LIB


if __name__ == "__main__":
    print(build())
