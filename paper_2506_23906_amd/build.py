"""Builds libmmvseg.so (HIP, gfx950 only) next to this file with hipcc, and the argument marshalling of the binding
(_marshal.so, a CPython extension on torch's headers) with g++."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "csrc", "mmvseg.hip")
LIB = os.path.join(HERE, "libmmvseg.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
MARSHAL_SRC = os.path.join(HERE, "csrc", "marshal.cpp")
MARSHAL_LIB = os.path.join(HERE, "_marshal.so")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"),
]


def build(verbose: bool = False, extra: list[str] | None = None, out: str | None = None) -> str:
    """Compiles the library; `extra` adds compiler flags (-D tunables), `out` names another output file."""
    lib = out or LIB
    tmp = lib + ".tmp.%d" % os.getpid()
    cmd = [HIPCC] + FLAGS + (extra or []) + ["-o", tmp, SRC]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature name; that note is harmless
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        sys.stderr.write(err + "\n")
        raise RuntimeError("hipcc failed building libmmvseg.so")
    if verbose and err.strip():
        sys.stderr.write(err + "\n")
    marshal = compile_marshal(verbose) if out is None else None
    os.replace(tmp, lib)              # (both are there before either is replaced)
    if marshal:
        os.replace(marshal, MARSHAL_LIB)
    return lib


def compile_marshal(verbose: bool = False) -> str:
    """Compiles the argument marshalling (host code only) against the installed torch; returns the file made."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    tmp = MARSHAL_LIB + ".tmp.%d" % os.getpid()
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM", "-DMMV_TORCH_VERSION=\"%s\"" % torch.__version__,
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-I", os.path.join(ROOT, "include"),
           "-isystem", sysconfig.get_paths()["include"], "-isystem", "/opt/rocm/include"]
    for path in cpp_extension.include_paths():
        cmd += ["-isystem", path]
    cmd += ["-o", tmp, MARSHAL_SRC, "-L" + libs, "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stderr + "\n")
        raise RuntimeError("g++ failed building _marshal.so")
    if verbose and res.stderr.strip():
        sys.stderr.write(res.stderr + "\n")
    return tmp


if __name__ == "__main__":
    print(build(verbose=True))
