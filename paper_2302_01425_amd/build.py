"""Builds in-tree: the HIP library (gfx950) with hipcc, csrc/*.hip -> lib/libsparse_topk.so, and the native call path of
the binding with the host compiler, csrc/host/call.cpp -> lib/_call.so."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIBDIR, "libsparse_topk.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


CALL_SRC = os.path.join(CSRC, "host", "call.cpp")
CALL_LIB = os.path.join(LIBDIR, "_call.so")


def call_command():
    """Host C++ against the headers of the torch that is installed; its libraries are found by name among those that it
    has loaded."""
    import torch
    home = os.path.dirname(torch.__file__)
    inc = os.path.join(home, "include")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
            "-Wno-sign-compare", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f'-DTOPK_TORCH_VERSION="{torch.__version__}"',
            "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
            "-isystem", sysconfig.get_paths()["include"], CALL_SRC, "-o", CALL_LIB,
            "-L" + os.path.join(home, "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python"]


def build_call(verbose: bool = True) -> bool:
    """Compile the native call path.  The binding works without it, so a failure (no host compiler, other torch headers)
    is reported and leaves none behind, not one of an earlier build either."""
    os.makedirs(LIBDIR, exist_ok=True)
    if os.path.exists(CALL_LIB):
        os.remove(CALL_LIB)
    try:
        cmd = call_command()
        if verbose:
            print(" ".join(cmd), flush=True)
        done = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        why, ok = done.stdout.strip(), done.returncode == 0
    except (ImportError, AttributeError, OSError) as e:
        why, ok = repr(e), False
    if why and (verbose or not ok):
        print(why, file=sys.stdout if ok else sys.stderr, flush=True)
    if not ok:
        print(f"WARNING: {CALL_SRC} was not built; calls take the Python path", file=sys.stderr, flush=True)
    return ok


def build_library(verbose: bool = True) -> str:
    """Compile every translation unit and link the shared library, then the native call path.  Always recompiles."""
    os.makedirs(LIBDIR, exist_ok=True)
    objs = []
    procs = []
    for src in sources():
        obj = os.path.join(LIBDIR, os.path.basename(src)[:-4] + ".o")
        cmd = [HIPCC, *FLAGS, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                                            text=True)))
        objs.append(obj)
    failed = False
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if out.strip() and verbose:
            print(out, flush=True)
        if pr.returncode != 0:
            failed = True
            print(f"FAILED: {src}", file=sys.stderr)
    if failed:
        raise RuntimeError("hipcc failed")
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    build_call(verbose)
    return LIB


if __name__ == "__main__":
    build_library()
