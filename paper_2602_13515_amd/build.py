"""Builds libspa2.so (HIP kernels + C ABI) for gfx950 and _operator.so (the operators' autograd functions) with hipcc, in-tree.

    python -m paper_2602_13515_amd.build          # compile everything, link the library
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libspa2.so")
OPERATOR = os.path.join(PKG, "_operator.so")
SOURCES = ["api.hip", "mask.hip", "fwd.hip", "bwd.hip", "bwd_dkdv.hip", "split.hip", "attention.hip", "backward.hip", "diag.hip", "distill.hip"]
# per-file flags: the dK/dV kernel mixes matrix products whose results the vector ALU reads (kept in ordinary
# registers by this option) with accumulators that it pins to the accumulation registers itself
EXTRA = {"bwd_dkdv.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 VALU forms are kept off (the compiler must not fuse float pairs)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    # raw_copy16_to_lds names m0 as clobbered (it is how the LDS address of a direct copy is passed)
    "-Wno-inline-asm",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(src: str, extra=()) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _operator_commands():
    """Compile and link lines of the operators' native code (host code over PyTorch's C++ API and libspa2.so)."""
    import torch
    from torch.utils import cpp_extension as ce
    obj = os.path.join(BUILD, "operator.o")
    compile_ = [HIPCC, "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                "-DTORCH_EXTENSION_NAME=_operator", "-DTORCH_API_INCLUDE_EXTENSION_H",
                f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-Wno-unused-command-line-argument",
                "-I", os.path.join(ROOT, "include"), "-I", sysconfig.get_paths()["include"]]
    for d in (*ce.include_paths(), os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include")):
        compile_ += ["-isystem", d]
    compile_ += ["-c", os.path.join(CSRC, "operator.cpp"), "-o", obj]
    link = [HIPCC, "-shared", "-fPIC", obj, "-o", OPERATOR, "-Wl,-rpath,$ORIGIN", LIB]
    for d in ce.library_paths():
        link += ["-L", d]
    link += ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch", "-ltorch_python"]
    return compile_, link


def _run(cmd, what: str) -> None:
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{r.stderr}")


def build(verbose: bool = True, extra=()) -> str:
    os.makedirs(BUILD, exist_ok=True)
    op_compile, op_link = _operator_commands()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        op = ex.submit(_run, op_compile, "hipcc on operator.cpp")
        objs = list(ex.map(lambda s: _compile(s, extra), SOURCES))
        op.result()
    # (the library's name in the operator's list of needed libraries is found next to it)
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-soname,libspa2.so", *objs, "-o", LIB], "link")
    _run(op_link, "link of the operators")
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(extra=tuple(sys.argv[1:]))
