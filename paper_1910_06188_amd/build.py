"""Build libq8.so (the C-ABI HIP library) in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libq8.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["q8_api.hip", "q8_elementwise.hip", "q8_gemm.hip", "q8_embedding.hip",
           "q8_gemm_tile_256x256_w4.hip", "q8_gemm_tile_256x256_w8.hip", "q8_gemm_tile_128x128_w4.hip",
           "q8_gemm_tile_192x256_w4.hip", "q8_gemm_tile_192x256_w8.hip", "q8_gemm_tile_192x128_w4.hip", "q8_layernorm.hip", "q8_attention.hip", "q8_ceiling.hip", "q8_fc_small.hip", "q8_gemm_direct.hip",
           "q8_gemm_tile_64x64_w4.hip", "q8_gemm_ring_64x64_s2.hip", "q8_gemm_ring_64x64_s3.hip",
           "q8_gemm_ring_128x64_s2.hip", "q8_gemm_ring_128x128_s1.hip", "q8_gemm_ring_192x128_s1.hip"]
OBJ_DIR = os.path.join(HERE, "_build")

# -ffp-contract=off: the product x*S of Eq. 1 must be rounded on its own before the
# rounding step.  Packed fp32 instructions are switched off for the whole library.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
         "-I", INCLUDE, "-I", CSRC]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err)


def build_binding(verbose: bool = False) -> str:
    """The Python entry points (csrc/binding.cpp), linked against libq8.so and this interpreter's torch."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    inc, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    abi = int(torch._C._GLIBCXX_USE_CXX11_ABI)
    _run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-D_GLIBCXX_USE_CXX11_ABI={abi}",
          "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), "-I", INCLUDE, "-isystem", inc,
          "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-I", sysconfig.get_paths()["include"],
          os.path.join(CSRC, "binding.cpp"), "-o", BINDING, LIB, "-L", lib, "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10",
          "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + lib], verbose)
    return BINDING


def build(verbose: bool = False) -> str:
    """Compile every translation unit (in parallel) and link libq8.so.  Always recompiles."""
    from concurrent.futures import ThreadPoolExecutor
    os.makedirs(OBJ_DIR, exist_ok=True)
    cc = hipcc()
    objs = [os.path.join(OBJ_DIR, s.replace(".hip", ".o")) for s in SOURCES]
    jobs = [[cc, *FLAGS, "-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
    with ThreadPoolExecutor(max_workers=min(8, len(jobs))) as ex:
        list(ex.map(lambda c: _run(c, verbose), jobs))
    _run([cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-soname,libq8.so", "-o", LIB, *objs], verbose)
    build_binding(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
