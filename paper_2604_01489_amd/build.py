"""Build step: compile the HIP sources into ``libgemm_epilogue.so`` (the operator) and
``libge_probes.so`` (the measurement probes) for gfx950, and the binding's argument marshalling into
an extension module of this interpreter.

``python -m paper_2604_01489_amd.build`` or ``build_library()``.  hipcc cross
compiles without a GPU.  The library is kept in-tree, next to this file.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgemm_epilogue.so")
PROBES_LIB = os.path.join(HERE, "libge_probes.so")
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
MARSHAL_STAMP = os.path.join(HERE, "_build", "marshal_torch_version")
MARSHAL_SOURCE = os.path.join(CSRC, "py_marshal.cpp")
# the longest compiles first (the pool takes the sources in this order)
LIB_SOURCES = ["conv_halo_14_11.hip", "conv_halo_12_12.hip", "conv_api.hip", "gemm_fused_t256.hip", "gemm_fused_t256_edge.hip", "gemm_fused_t256_kedge.hip", "gemm_fused_t128.hip",
               "gemm_fused_t128_edge.hip", "gemm_fused_t128_kedge.hip",
               "gemm_fused_w4_e0.hip", "gemm_fused_w4_e1.hip", "gemm_fused_w4_e2.hip", "gemm_epilogue_api.hip",
               "gemm_tile64.hip", "gemm_tile64_short.hip", "gemm_tile64_conv.hip", "gemm_small.hip", "gemm_ragged_t128.hip", "gemm_ragged_t128_w8.hip", "gemm_ragged_t64.hip", "gemm_fused_api.hip", "gemm_symm_api.hip", "gemm_diag.hip", "gemm_rowsum.hip"]
PROBE_SOURCES = ["ge_probes.hip"]
SOURCES = LIB_SOURCES + PROBE_SOURCES
# packed fp32 instructions are kept off: some of their forms have misbehaved on this hardware
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _includes(path, seen):
    """Files a source pulls in through #include "..." (transitively)."""
    import re
    if path in seen or not os.path.exists(path):
        return seen
    seen.add(path)
    for inc in re.findall(r'^\s*#include\s+"([^"]+)"', open(path).read(), flags=re.M):
        _includes(os.path.normpath(os.path.join(os.path.dirname(path), inc)), seen)
    return seen


def _newer(built, deps):
    return os.path.exists(built) and all(os.path.getmtime(d) <= os.path.getmtime(built) for d in deps)


def build_marshal(verbose: bool = False) -> str:
    """The extension module: host code only, against torch's headers and the libraries that ``import torch`` loads, and for that torch alone."""
    import torch
    top = os.path.dirname(torch.__file__)
    os.makedirs(os.path.dirname(MARSHAL_STAMP), exist_ok=True)
    lib = os.path.join(top, "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           f'-DGE_TORCH_VERSION="{torch.__version__}"',
           "-I" + sysconfig.get_paths()["include"], "-isystem", os.path.join(top, "include"), "-o", MARSHAL, MARSHAL_SOURCE,
           "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath," + lib]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("g++ failed on py_marshal.cpp")
    with open(MARSHAL_STAMP, "w") as f:
        f.write(torch.__version__)
    return MARSHAL


def marshal_is_current() -> bool:
    """Newer than what it is compiled from, and for the torch that is installed (as the build noted: a module that is loaded to be asked stays loaded)."""
    import torch
    return (_newer(MARSHAL, _includes(MARSHAL_SOURCE, set())) and os.path.exists(MARSHAL_STAMP) and
            open(MARSHAL_STAMP).read() == torch.__version__)


def build_library(verbose: bool = False, extra_flags=(), incremental: bool = False) -> str:
    """Compile every source to an object (in parallel: the kernel templates dominate the build
    time), then link the two libraries.  ``incremental`` keeps the objects that are newer than
    the source and every header it includes (for work on one file; the default compiles all)."""
    from concurrent.futures import ThreadPoolExecutor
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]

    def compile_one(src):
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        if incremental and not extra_flags and _newer(obj, _includes(os.path.join(CSRC, src), set())):
            return obj
        cmd = ["hipcc", *compile_flags, *extra_flags, "-c", "-o", obj, os.path.join(CSRC, src)]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError(f"hipcc failed on {src}")
        return obj

    def marshal():
        if incremental and marshal_is_current():
            return
        try:
            build_marshal(verbose)
        except (OSError, RuntimeError) as err:       # no g++, or no headers: the library is whole without it
            if os.path.exists(MARSHAL):
                os.remove(MARSHAL)
            sys.stderr.write(f"{err}\nno native marshalling: the binding's Python code takes every call\n")

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as pool:
        marshalled = pool.submit(marshal)
        objs = list(pool.map(compile_one, SOURCES))
        marshalled.result()
    n = len(LIB_SOURCES)
    for out, group in ((LIB, objs[:n]), (PROBES_LIB, objs[n:])):
        cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out, *group]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError("link failed")
    return LIB


def library_is_current() -> bool:
    """Whether the two HIP libraries are newer than the sources that each is made of."""
    def deps(sources):
        seen = set()
        for src in sources:
            _includes(os.path.join(CSRC, src), seen)
        return seen
    return _newer(LIB, deps(LIB_SOURCES)) and _newer(PROBES_LIB, deps(PROBE_SOURCES))


if __name__ == "__main__":
    print(build_library(verbose=True, incremental="--incremental" in sys.argv[1:]))
