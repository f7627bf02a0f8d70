"""Compile the HIP library (hipcc, gfx950) and the binding's native calls in-tree.  `python -m paper_1910_00178_amd.build`."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "csrc", "ngemm.hip")
LIB = os.path.join(HERE, "libngemm.so")
CALLS_SRC = os.path.join(HERE, "csrc", "calls.c")
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "--offload-arch=gfx950",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=off", "-fPIC", "-shared", "-std=c++17",
    "-I" + os.path.join(ROOT, "include"),
    "-Wall", "-Wextra", "-Wno-pass-failed",
    "-Wl,--no-undefined",        # a kernel the host pass failed to emit must fail the build, not the first load
]


CC = os.environ.get("CC", "gcc")
CALLS_FLAGS = ["-O2", "-std=gnu11", "-fPIC", "-shared", "-Wall", "-Wextra", "-Wno-cast-function-type", "-Wno-missing-field-initializers",
               "-I" + sysconfig.get_path("include")]


def _compile(cmd, src, lib, verbose):
    cmd = [*cmd, "-o", lib, src]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(cmd[0] + " failed:\n" + out)
    if verbose and out.strip():
        print(out)
    return lib


def build_library(verbose=False):
    """The HIP library, and the binding's native calls beside it."""
    _compile([CC, *CALLS_FLAGS], CALLS_SRC, CALLS, verbose)
    return _compile([HIPCC, *FLAGS], SRC, LIB, verbose)


if __name__ == "__main__":
    print(build_library(verbose=True))
    sys.exit(0)
