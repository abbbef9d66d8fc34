"""Build the HIP library (csrc/*.hip -> libzc.so) for gfx950 with hipcc, and the native calls of the binding for this Python, in-tree."""
import os
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libzc.so")
SOURCES = ["zc_api.hip"]
CALLS = os.path.join(HERE, "_zc_calls" + sysconfig.get_config_var("EXT_SUFFIX"))      # (named for this Python: another one leaves it alone)

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC", "-shared",
    "-ffp-contract=off",                                     # quantisation is defined by separate roundings
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-kernarg-preload-count=16",            # a kernel's leading scalar arguments are in registers when a wave starts
    "-Wall", "-Wno-unused-function",
]


def build(verbose=False, extra=()):
    cmd = ["hipcc", *FLAGS, *extra, *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    build_calls(verbose)
    return LIB


def build_calls(verbose=False):
    """The native calls, which the binding does without where they are missing: they need the headers of this Python and a C++ compiler."""
    include = sysconfig.get_paths()["include"]
    if os.path.exists(CALLS):
        os.remove(CALLS)                                     # (not one of other sources beside the library)
    if not os.path.exists(os.path.join(include, "Python.h")) or not shutil.which("g++"):
        print("no headers of this Python or no g++: the binding goes through ctypes alone")
        return
    cmd = ["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I" + include, os.path.join(CSRC, "zc_calls.cpp"), "-o", CALLS]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)


if __name__ == "__main__":
    print(build(verbose=True))
