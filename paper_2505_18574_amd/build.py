"""Build in-tree: csrc/*.hip + api.cpp -> libac_mi355x.so (the HIP library, gfx950 only), csrc/binding.cpp -> _binding.so
(the compiled side of ops.py, host code against this interpreter's torch)."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libac_mi355x.so")
BINDING = os.path.join(HERE, "_binding.so")

SOURCES = ["api.cpp", "gemm_i8.hip", "gemm_i8_trans.hip", "conv_direct.hip", "gemm_bf16.hip", "batched_f32.hip", "tinympc_f32.hip"]

# Packed-fp32 VALU forms are switched off for every device compile.
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj] + COMMON + DEVICE_FLAGS
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    return obj


def _build_binding() -> None:
    """Needs LIB, which the binding finds beside itself, before any in LD_LIBRARY_PATH.  It is linked by name: a path would be
    recorded, and followed from a copy of the package too.  torch's own libraries are in the process before it is loaded."""
    import torch

    root = os.path.dirname(torch.__file__)
    include = [os.path.join(root, "include"), sysconfig.get_paths()["include"], os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] + [f"-I{i}" for i in include]
    cmd += [os.path.join(CSRC, "binding.cpp"), "-o", BINDING, "-L" + HERE, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN,--disable-new-dtags", "-L" + os.path.join(root, "lib"),
            "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"building the binding failed:\n{r.stderr}")


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [_hipcc(), "-shared", "-fPIC", "-o", LIB] + objs + ["--offload-arch=gfx950"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    _build_binding()
    if verbose:
        print("built", LIB, BINDING)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
