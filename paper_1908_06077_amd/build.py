"""Build libnuq.so (the C-ABI library) in-tree with hipcc for gfx950, and _nuq_calls.so (its calls from Python) with g++."""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "nuq.hip")
LIB = os.path.join(HERE, "libnuq.so")
CALLS_SRC = os.path.join(HERE, "csrc", "nuq_calls.cpp")
CALLS = os.path.join(HERE, "_nuq_calls.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-shared", "-fPIC",
]


def _calls_command(out: str) -> list[str]:
    torch = list(importlib.util.find_spec("torch").submodule_search_locations)[0]      # found, not imported
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=1",
            "-I" + os.path.join(torch, "include"), "-I" + os.path.join(torch, "include", "torch", "csrc", "api", "include"),
            "-I" + sysconfig.get_paths()["include"], "-o", out, CALLS_SRC,
            "-L" + os.path.join(torch, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp, calls_tmp = ("%s.tmp.%d" % (x, os.getpid()) for x in (LIB, CALLS))
    running = [(what, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
               for what, cmd in (("hipcc", [hipcc, *HIPCC_FLAGS, "-o", tmp, SRC]), ("g++", _calls_command(calls_tmp)))]
    failed = []
    for what, p in running:
        try:
            out = p.communicate(timeout=900)[0]
        except subprocess.TimeoutExpired:
            p.kill()
            out = p.communicate()[0]
        if p.returncode != 0:
            failed.append("%s failed:\n%s" % (what, out))
        elif verbose and out:
            print(out)
    if failed:
        raise RuntimeError("\n".join(failed))
    os.replace(tmp, LIB)
    os.replace(calls_tmp, CALLS)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
