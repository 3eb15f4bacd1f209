"""Compile the HIP library for gfx950 into paper_2508_06041_amd/libdpllm.so and the binding's native part into _calls.so (in-tree)."""
import os
import re
import subprocess
import sys
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


def spilled(report: str) -> list:
    """The kernels that keep vector registers in scratch memory, from what the compiler says about the resources of each: their code is
    written for the registers there are, and one that does not fit makes every launch of it slower without any other sign."""
    kernels = []
    for part in report.split("Function Name: ")[1:]:
        used = {k: int(v) for k, v in re.findall(r"(ScratchSize|VGPRs Spill)[^:\n]*: (\d+)", part)}
        if any(used.values()):
            kernels.append(part.split()[0])
    return kernels


def build(verbose: bool = False, extra=()) -> str:
    cmd = ["/opt/rocm/bin/hipcc", *FLAGS, *extra, "-o", LIB] + [os.path.join(CSRC, s) for s in SOURCES]
    calls = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra", "-I" + sysconfig.get_paths()["include"], "-o", CALLS,
             os.path.join(CSRC, "py_calls.cpp")]
    for c in (calls, cmd + ["-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics"]):
        if verbose:
            print(" ".join(c))
        done = subprocess.run(c, stderr=subprocess.PIPE, text=True)
        sys.stderr.write("".join(line for line in done.stderr.splitlines(True) if "[-Rpass-analysis" not in line and not line.startswith("In file included")))
        done.check_returncode()
    if spilled(done.stderr):
        raise RuntimeError("vector registers spilled: " + ", ".join(spilled(done.stderr)))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
