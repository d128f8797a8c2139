"""Builds liblbpwht.so (HIP kernels + C ABI) for gfx950 with hipcc and the CPython module _native.so
(csrc/native.cpp, the binding's fast path; host code only, compiled with g++ against torch's headers), in-tree.

    python -m paper_2309_15275_amd.build          # compile everything, link
"""
import concurrent.futures
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "liblbpwht.so")
NATIVE = os.path.join(PKG, "_native.so")

SOURCES = ["lbp_host.cpp", "wht_kernels.hip", "wht_mfma_kernels.hip", "energy_kernels.hip", "extra_kernels.hip", "bias_kernels.hip", "gemm_kernels.hip", "gemm_f32_mfma.hip", "gemm_mfma.hip",
           "gemm_mfma_128x128.hip", "gemm_mfma_64x128.hip", "gemm_mfma_128x256.hip",
           "gemm_mfma_256x256.hip", "gemm_mfma_64x64.hip", "gemm_mfma_256x192.hip", "gemm_mfma_256x128.hip", "gemm_mfma_pair.hip", "gemm_mfma_pair_deep.hip", "gemm_mfma_pair_wide.hip",
           "lbp_api.hip"]

# -packed-fp32-ops off: the compiler must not form packed fp32 instructions on this target.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", "-x", "hip"] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _run(cmd, what):
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{res.stderr}")


def _compile_native():
    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    obj = os.path.join(BUILD, "native.o")
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem", inc,
          "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
          "-isystem", sysconfig.get_paths()["include"], "-c", os.path.join(CSRC, "native.cpp"), "-o", obj], "native.cpp")
    return obj


def _link_native(obj):
    import torch
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    _run(["g++", "-shared", obj, "-o", NATIVE, "-L" + lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python",
          "-L" + PKG, "-llbpwht", "-Wl,-rpath,$ORIGIN"], "linking _native.so")


def build(verbose=True):
    """Compiles every source (always) and links both shared objects.  Returns the library's path."""
    os.makedirs(BUILD, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=8) as pool:
        native = pool.submit(_compile_native)
        objs = list(pool.map(_compile, SOURCES))
        native_obj = native.result()
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    _link_native(native_obj)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
