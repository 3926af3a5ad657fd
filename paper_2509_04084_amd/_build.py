"""Builds the HIP library in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "liblowdiff.so")
SOURCES = ["ld_api.hip", "ld_config.hip", "ld_merge_sparse.hip", "ld_recover.hip", "ld_check_diff.hip", "ld_merge_sparse_adam.hip", "ld_combine_sparse.hip", "ld_dense.hip", "ld_compress.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


MARSHAL = os.path.join(PKG, "_marshal.so")


def build_marshal(force: bool = True) -> str:
    """Compiles the binding's argument marshalling (a CPython module against torch's headers); returns its path."""
    src = os.path.join(CSRC, "ld_marshal.cpp")
    if not force and os.path.exists(MARSHAL) and os.path.getmtime(MARSHAL) >= os.path.getmtime(src):
        return MARSHAL
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    base = os.path.dirname(torch.__file__)
    tmp = f"{MARSHAL}.{os.getpid()}.tmp"  # ranks that build at once must not write into each other's file
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DLD_BUILT_FOR_TORCH="{torch.__version__}"']
    cmd += ["-isystem" + d for d in cpp_extension.include_paths()] + ["-I", sysconfig.get_paths()["include"]]
    cmd += [src, "-o", tmp, "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed building _marshal.so\n" + res.stdout + res.stderr)
    os.replace(tmp, MARSHAL)
    return MARSHAL


def build_library(force: bool = True, verbose: bool = False) -> str:
    """Compiles every HIP source into liblowdiff.so; returns its path."""
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    deps = srcs + [os.path.join(CSRC, "ld_common.h"), os.path.join(CSRC, "ld_sparse_common.h"), os.path.join(CSRC, "ld_thin.h"),
                   os.path.join(CSRC, "ld_map.h"), os.path.join(CSRC, "ld_combine_shape.h"),
                   os.path.join(ROOT, "include", "lowdiff.h")]
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in deps):
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = f"{LIB}.{os.getpid()}.tmp"
    cmd = [hipcc] + FLAGS + ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", tmp] + srcs
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(res.stdout)
        print(res.stderr)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed building liblowdiff.so")
    os.replace(tmp, LIB)
    return LIB
