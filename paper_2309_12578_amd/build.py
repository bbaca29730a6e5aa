"""Build libspion.so (HIP, gfx950 only) with hipcc and the front end's call path (_spion_host.so, host code
against torch's C++ headers) with g++, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libspion.so")
HOST = os.path.join(HERE, "_spion_host.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          # No compiler-generated packed-fp32 instructions (v_pk_add/mul/fma_f32).  The feature belongs
          # to the gfx950 pass, which honours it (a float2 fused multiply-add compiles to one
          # v_pk_fma_f32 without the flag and to two v_fma_f32 with it); hipcc also hands the flag to
          # its host pass, which prints "'-packed-fp32-ops' is not a recognized feature for this
          # target" once per source.  That line is left in the compiler output.
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# (source, extra flags).  The pattern kernels take threshold decisions in fp64 whose rounding must
# follow the sequential definition: no fused multiply-add contraction there.
SOURCES = [
    ("spion_api.hip", ["-ffp-contract=off"]),
    ("pattern_kernels.hip", ["-ffp-contract=off"]),
    ("producer_kernels.hip", []),
    # MFMA accumulators in ordinary VGPRs: the softmax between two products reads them with VALU
    # instructions, and the AGPR form costs a register copy per value per step
    ("attn_kernels.hip", ["-mllvm", "-amdgpu-mfma-vgpr-form"]),
    ("attn_bf16_kernels.hip", ["-mllvm", "-amdgpu-mfma-vgpr-form"]),
    ("attn_bwd_bf16_kernels.hip", ["-mllvm", "-amdgpu-mfma-vgpr-form"]),
    ("norm_kernels.hip", []),
    ("projection_kernels.hip", ["-mllvm", "-amdgpu-mfma-vgpr-form"]),
]


def host_object() -> str:
    """Compile csrc/host_ext.cpp (no GPU code)."""
    import torch
    root = os.path.dirname(torch.__file__)
    obj = os.path.join(CSRC, "host_ext.o")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I" + sysconfig.get_paths()["include"], "-isystem", os.path.join(root, "include"), "-isystem",
           os.path.join(root, "include", "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
           "-c", os.path.join(CSRC, "host_ext.cpp"), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed for host_ext.cpp:\n" + res.stderr)
    return obj


def link_host(obj: str) -> None:
    import torch
    cmd = ["g++", "-shared", "-o", HOST, obj, LIB, "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"),
           "-ltorch_python", "-ltorch", "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link of _spion_host.so failed:\n" + res.stderr)


def build(verbose: bool = False) -> str:
    """Compile every source and link the two shared libraries; always recompiles."""
    objs = []

    def compile_one(item):
        src, extra = item
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [HIPCC, *COMMON, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        res = subprocess.run(cmd, capture_output=True, text=True)
        err = res.stderr
        if res.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        host = ex.submit(host_object)
        objs = list(ex.map(compile_one, SOURCES))
        host = host.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-soname,libspion.so", "-o", LIB, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    link_host(host)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
