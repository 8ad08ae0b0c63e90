"""Build libeagletv.so (hipcc, gfx950) and its Python binding in-tree.  Run as ``python -m paper_2603_08088_amd.build``."""
from __future__ import annotations

import importlib.util
import os
import runpy
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
GENERATED = os.path.join(CSRC, "_build")   # what the scripts of csrc write for the compiler
LIB = os.path.join(HERE, "libeagletv.so")
PROBE_LIB = os.path.join(HERE, "libeagletv_probe.so")   # measurement aids (include/eagletv_probe.h), separate on purpose
BINDING = os.path.join(HERE, "_binding.so")   # the calls of the library as a Python module (csrc/binding.cpp), host code only
SOURCES = ["api.hip", "mask.hip", "attention.hip", "posterior.hip", "commit.hip", "lmhead.hip", "branch.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=14",   # a kernel's leading scalar arguments are in registers when it starts
         "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", GENERATED]


def _hipcc(sources, target, verbose, extra=()):
    # extern "C" entry points are exported explicitly; everything else stays hidden
    _run([HIPCC] + FLAGS + ["-DETV_BUILDING"] + list(extra) + [os.path.join(CSRC, s) for s in sources] + ["-o", target], verbose)


def _host_binding(verbose):
    """The Python binding.  It needs torch, its headers, Python's and a C++ compiler; the C library is complete without it."""
    cxx = os.environ.get("CXX", "g++").split()
    py_include, missing = sysconfig.get_paths()["include"], []
    if shutil.which(cxx[0]) is None:
        missing.append(cxx[0])
    if not os.path.exists(os.path.join(py_include, "Python.h")):
        missing.append("Python.h")
    spec = importlib.util.find_spec("torch")
    torch_dir = os.path.dirname(spec.origin) if spec else None
    if torch_dir is None or not os.path.exists(os.path.join(torch_dir, "include", "ATen", "ATen.h")):
        missing.append("torch")
    if missing:
        if os.path.exists(BINDING):
            os.remove(BINDING)   # one of another library must not stay
        print(f"{os.path.basename(BINDING)}, which Python calls need, is not built: no {', '.join(missing)}", flush=True)
        return
    import torch
    from torch.utils import cpp_extension
    torch_lib = os.path.join(torch_dir, "lib")
    # HIP's headers: beside the compiler, which HIPCC may name by its path or as a command
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(shutil.which(HIPCC) or HIPCC)))
    includes = [os.path.join(ROOT, "include"), py_include, os.path.join(rocm, "include")] + cpp_extension.include_paths()
    _run(cxx + ["-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] + [f"-I{d}" for d in includes] +
         [os.path.join(CSRC, "binding.cpp"), "-o", BINDING, f"-L{HERE}", f"-L{torch_lib}", "-l:libeagletv.so", "-lc10", "-lc10_hip", "-ltorch_cpu",
          "-ltorch_python", "-Wl,-rpath,$ORIGIN"], verbose)


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + out)
    if verbose and out.strip():
        print(out)


def _generate():
    os.makedirs(GENERATED, exist_ok=True)
    text = runpy.run_path(os.path.join(CSRC, "attn_wide_loop.py"))["header"]()
    with open(os.path.join(GENERATED, "attn_wide_loop.h"), "w") as f:
        f.write(text)


def build(verbose: bool = False, extra=()) -> str:
    _generate()
    _hipcc(SOURCES, LIB, verbose, extra)
    _hipcc(["probe.hip"], PROBE_LIB, verbose)
    _host_binding(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
