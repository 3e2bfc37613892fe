"""Builds libcure.so in-tree for gfx950 with hipcc, and beside it the extension
module _native.so, the Python binding's argument marshalling, with the host compiler.

Usage: python -m paper_2608_00531_amd.build   (or call build_library()).
"""

import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB_DIR = os.path.join(PKG, "_lib")
LIB_PATH = os.path.join(LIB_DIR, "libcure.so")
NATIVE_PATH = os.path.join(LIB_DIR, "_native.so")
INCLUDE = os.path.join(ROOT, "include")

SOURCES = ["api.cpp", "margins.hip", "accept.hip", "tree_attn.hip", "repair.hip", "commit.hip", "ceiling.hip"]

# Packed fp32 arithmetic is disabled for all device code.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc():
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def _run(cmd, out, verbose):
    """Runs a compiler that writes out + ".tmp", then moves the result into place."""
    cmd = cmd + ["-o", out + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass warns that it does not know the packed-fp32 feature.
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (os.path.basename(cmd[0]), err))
    if verbose and err.strip():
        print(err, file=sys.stderr)
    os.replace(out + ".tmp", out)


def build_native(verbose=False):
    """The binding's extension module: links libcure.so (beside it) and torch."""
    import torch
    from torch.utils import cpp_extension
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           "-I", INCLUDE, "-isystem", sysconfig.get_paths()["include"]]
    for path in cpp_extension.include_paths("cuda"):
        cmd += ["-isystem", path]
    cmd += [os.path.join(CSRC, "binding.cpp"), "-L" + LIB_DIR, "-lcure", "-Wl,-rpath,$ORIGIN",
            "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"),
            "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    _run(cmd, NATIVE_PATH, verbose)
    return NATIVE_PATH


def build_library(verbose=False):
    os.makedirs(LIB_DIR, exist_ok=True)
    _run([hipcc()] + HIPCC_FLAGS + ["-I", INCLUDE, "-I", CSRC] +
         [os.path.join(CSRC, s) for s in SOURCES], LIB_PATH, verbose)
    build_native(verbose)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
