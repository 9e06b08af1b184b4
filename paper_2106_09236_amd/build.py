"""Build libprobsparse.so (HIP kernels for gfx950 + the C-ABI host code) and the Python module _native (the hot
entry points for tensors, on top of that library; calls take ctypes where it is missing) in-tree.

    python -m paper_2106_09236_amd.build

Cross-compiles without a GPU.  The library lands next to this file so that it
travels with the source tree.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(CSRC, "_build")
LIB_PATH = os.path.join(HERE, "libprobsparse.so")

NATIVE_PATH = os.path.join(HERE, "_native.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-I", os.path.join(HERE, "..", "include")]
# packed-FP32 instructions are switched off for device code on purpose
DEVICE = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *COMMON, *DEVICE, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_library(verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", LIB_PATH, *objs,
           "-Wl,-rpath,/opt/rocm/lib", "-Wl,--no-undefined", "-Wl,-soname,libprobsparse.so"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print(f"built {LIB_PATH} from {len(srcs)} sources")
    return LIB_PATH


def build_native(verbose: bool = True) -> str:
    """The extension module: host code only, against the installed torch's headers and libprobsparse.so."""
    import torch
    root = os.path.dirname(torch.__file__)
    inc = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
           sysconfig.get_paths()["include"], "/opt/rocm/include"]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(f for i in inc for f in ("-isystem", i)),
           os.path.join(CSRC, "python", "psa_native.cpp"), "-o", NATIVE_PATH, "-L" + os.path.join(root, "lib"),
           "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-L" + HERE, "-lprobsparse", "-Wl,-rpath,$ORIGIN", "-Wl,-soname,_native.so"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("building _native failed:\n" + r.stderr)
    if verbose:
        print(f"built {NATIVE_PATH}")
    return NATIVE_PATH


if __name__ == "__main__":
    build_library()
    try:
        build_native()
    except (RuntimeError, OSError) as e:    # no host compiler, say: the library is usable without the module
        sys.stderr.write(f"{e}\nthe Python entry points will go through ctypes\n")
