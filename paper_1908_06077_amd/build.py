"""Build libnuq.so (the C-ABI library) in-tree with hipcc for gfx950, and _nuq_calls.so (its calls from Python) with g++."""
from __future__ import annotations

import hashlib
import os
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "nuq.hip")
LIB = os.path.join(HERE, "libnuq.so")
CALLS_SRC = os.path.join(HERE, "csrc", "nuq_calls.cpp")
CALLS = os.path.join(HERE, "_nuq_calls" + sysconfig.get_config_var("EXT_SUFFIX"))       # it serves one Python only, and one torch
HEADER = os.path.join(os.path.dirname(HERE), "include", "nuq.h")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-shared", "-fPIC",
]


def _header_key() -> str:
    """A number that stands for the interface: both files carry it, and the binding refuses a pair that differs."""
    with open(HEADER, "rb") as f:
        return "-DNUQ_HEADER_KEY=0x%sull" % hashlib.sha256(f.read()).hexdigest()[:16]


def _calls_command(out: str) -> list[str]:
    import torch
    root = os.path.dirname(torch.__file__)
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", _header_key(),
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(), '-DNUQ_TORCH_VERSION="%s"' % torch.__version__,
            "-I" + os.path.join(root, "include"), "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
            "-I" + sysconfig.get_paths()["include"], "-o", out, CALLS_SRC,
            "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp, calls_tmp = ("%s.tmp.%d" % (x, os.getpid()) for x in (LIB, CALLS))
    commands = (("hipcc", [hipcc, *HIPCC_FLAGS, _header_key(), "-o", tmp, SRC]), ("g++", _calls_command(calls_tmp)))
    for what, cmd in commands:                         # before either runs
        if not shutil.which(cmd[0]):
            raise RuntimeError("no %s: %s does not exist" % (what, cmd[0]))
    running = [(what, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
               for what, cmd in commands]
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
