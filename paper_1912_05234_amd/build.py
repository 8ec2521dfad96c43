"""Builds the gfx950 shared library from csrc/*.hip with hipcc (cross-compiles without a GPU), and the extension
module of the Python calls over it from csrc/torch_calls.cpp.

    python -m paper_1912_05234_amd.build
"""
import glob
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libcnn_mi355x.so")
CALLS = os.path.join(PKG, "_calls.so")

# Packed fp32 VALU forms are switched off for device code on purpose (hipcc would
# otherwise form them from scalar float code).
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-Wno-unused-command-line-argument"]


def sources():
    return sorted(glob.glob(os.path.join(PKG, "csrc", "*.hip")))


def run(cmd, verbose):
    """cmd without its output file, which is made under a temporary name and moved into place."""
    target, cmd = cmd[0], cmd[1:]
    tmp = target + ".tmp%d" % os.getpid()
    cmd = cmd + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout)
        raise RuntimeError("%s failed (exit %d)" % (os.path.basename(cmd[0]), res.returncode))
    if verbose and res.stdout.strip():
        print(res.stdout)
    os.replace(tmp, target)


def build_calls(verbose=False):
    import torch
    root = os.path.dirname(torch.__file__)
    include = [os.path.join(ROOT, "include"), "/opt/rocm/include", os.path.join(root, "include"),
               os.path.join(root, "include", "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"]]
    run([CALLS, os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
         "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI] + ["-I" + d for d in include] +
        [os.path.join(PKG, "csrc", "torch_calls.cpp"), "-L" + os.path.join(root, "lib")] +
        ["-l" + n for n in ("torch_python", "torch_cpu", "torch_hip", "c10", "c10_hip")] +
        ["-L" + PKG, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN"], verbose)


def build(verbose=False, extra=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    run([LIB, hipcc] + HIPCC_FLAGS + list(extra) +
        ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")] + sources(), verbose)
    build_calls(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
