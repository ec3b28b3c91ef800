"""Builds the C-ABI library (csrc/*.hip -> lib/libpermuquant.so) for gfx950 with hipcc, and the binding of its hot calls
(csrc/pq_calls.cpp -> lib/_pq_calls.so).

Cross-compiles without a GPU.  Usage: `python -m paper_2605_09503_amd.build`.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(LIBDIR, "libpermuquant.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                 # the quantizer arithmetic is pinned op by op
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes",
]


# the Python binding of the hot calls (csrc/pq_calls.cpp): host code against this interpreter and its torch
CALLS = os.path.join(LIBDIR, "_pq_calls.so")


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str) -> str:
    obj = os.path.join(OBJDIR, src[:-4] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    warn = "\n".join(l for l in r.stderr.splitlines()
                     if "warning" in l and "packed-fp32-ops" not in l)
    if warn:
        sys.stderr.write(warn + "\n")
    return obj


def _build_calls() -> bool:
    """The binding; False, with a message, where what it is built with is missing: the library stands without it."""
    cxx, headers = os.environ.get("CXX", "g++"), sysconfig.get_paths()["include"]
    try:
        import torch
    except ImportError:
        torch = None
    missing = ("torch" if torch is None else
               "a host compiler (%s)" % cxx if shutil.which(cxx) is None else
               "the interpreter's headers (%s)" % headers if not os.path.exists(os.path.join(headers, "Python.h")) else None)
    if missing:
        if os.path.exists(CALLS):
            os.remove(CALLS)                 # one of another build
        sys.stderr.write("binding of the hot calls not built, %s is missing: %s goes without it\n" % (missing, LIB))
        return False
    root = os.path.dirname(torch.__file__)
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           "-I", headers, "-isystem", os.path.join(root, "include"),
           "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-isystem", os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"),
           os.path.join(CSRC, "pq_calls.cpp"), "-o", CALLS, "-Wall", "-L", LIBDIR, "-lpermuquant", "-Wl,-rpath,$ORIGIN",
           "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("building the binding failed:\n%s\n%s" % (r.stdout, r.stderr))
    return True


def build(verbose: bool = True) -> str:
    os.makedirs(LIBDIR, exist_ok=True)
    os.makedirs(OBJDIR, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    _build_calls()
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
