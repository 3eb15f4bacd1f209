"""Compile the HIP library for gfx950 into paper_2508_06041_amd/libdpllm.so and the binding's native part into _calls.so (in-tree)."""
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdpllm.so")
SOURCES = ["dpllm_api.hip"]
CALLS = os.path.join(HERE, "_calls.so")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unused-result",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # the first kernel arguments arrive in scalar registers with the launch instead of being loaded from memory
         "-mllvm", "-amdgpu-kernarg-preload-count=14"]


def build(verbose: bool = False, extra=()) -> str:
    cmd = ["/opt/rocm/bin/hipcc", *FLAGS, *extra, "-o", LIB] + [os.path.join(CSRC, s) for s in SOURCES]
    calls = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra", "-I" + sysconfig.get_paths()["include"], "-o", CALLS,
             os.path.join(CSRC, "py_calls.cpp")]
    for c in (calls, cmd):
        if verbose:
            print(" ".join(c))
        subprocess.run(c, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
