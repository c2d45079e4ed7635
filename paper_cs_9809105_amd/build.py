"""Build the C-ABI library ``libhs.so`` (HIP kernels for gfx950 + host API)
and the binding's native call path ``_hs_torch.so``.

    python -m paper_cs_9809105_amd.build [--verbose]

Compiles in-tree with hipcc; the result sits next to this file so that it
travels with the source tree.  Every build recompiles.

``build(out=..., extra=...)`` writes a variant elsewhere with extra flags
(the sanitized copy of the CPU test-suite); the product library is always
``libhs.so`` beside this file.
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhs.so")
NATIVE = os.path.join(HERE, "_hs_torch.so")     # the binding's native call path (csrc/hs_torch.cpp)
SOURCES = [os.path.join(CSRC, "hs_kernels.hip"), os.path.join(CSRC, "hs_wave.hip"),
           os.path.join(CSRC, "hs_prep.hip"), os.path.join(CSRC, "hs_nbody.hip"),
           os.path.join(CSRC, "hs_api.cpp"), os.path.join(CSRC, "hs_noalloc.hip")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed FP32 instructions are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    "-Wall", "-Wno-unused-function",
]


def build(verbose=False, extra=(), out=None):
    target = out or LIB
    tmp = target + ".tmp"
    cmd = [HIPCC] + FLAGS + list(extra) + SOURCES + ["-o", tmp]
    if verbose:
        cmd.insert(1, "-Rpass-analysis=kernel-resource-usage")
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    log = "\n".join(l for l in res.stdout.splitlines()
                    if "packed-fp32-ops' is not a recognized feature" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + log)
    os.replace(tmp, target)
    if verbose and log.strip():
        print(log)
    return target


def build_native():
    """Compile the Python module through which binding.py makes its calls."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = NATIVE + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(root, "include"),
           "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "hs_torch.cpp"), "-o", tmp, "-L", os.path.join(root, "lib"),
           "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10", "-lc10_hip"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stdout)
    os.replace(tmp, NATIVE)
    return NATIVE


if __name__ == "__main__":
    print(build(verbose="--verbose" in sys.argv))
    print(build_native())
