"""Compile the HIP library for gfx950, in-tree.

Produces ``libresbm.so`` (bf16 activations), ``libresbm_f32.so`` (the fp32
validation build) and ``_marshal.so`` (the binding's argument marshalling, host
code against torch's and CPython's C++ interfaces) next to this file.  Run ``python -m paper_2604_11947_amd.build``.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRC = os.path.join(PKG, "csrc", "resbm_kernels.hip")
SRC_MATRIX = os.path.join(PKG, "csrc", "resbm_matrix.hip")
SRC_TWO = os.path.join(PKG, "csrc", "resbm_two.hip")
DEPS = [SRC, SRC_MATRIX, SRC_TWO, os.path.join(PKG, "csrc", "resbm_buffer.hpp"), os.path.join(PKG, "csrc", "resbm_host.hpp"), os.path.join(PKG, "csrc", "resbm_mfma.hpp"), os.path.join(PKG, "csrc", "resbm_plan.hpp"),
        os.path.join(PKG, "csrc", "resbm_short.hpp"),
        os.path.join(ROOT, "include", "resbm.h")]

SRC_MARSHAL = os.path.join(PKG, "csrc", "resbm_marshal.cpp")
MARSHAL = os.path.join(PKG, "_marshal.so")

LIBS = {"bf16": "libresbm.so", "f32": "libresbm_f32.so"}


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build the HIP library)")


def command(variant: str, out: str) -> list[str]:
    cmd = [hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
           # packed fp32 VALU ops stay disabled in every HIP build of this library
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-o", out, SRC, SRC_MATRIX, SRC_TWO]
    if variant == "f32":
        cmd.insert(1, "-DRESBM_IO_F32_BUILD=1")
    return cmd


def marshal_command(out: str) -> list[str]:
    import sysconfig

    import torch

    root = os.path.dirname(torch.__file__)
    inc, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    return [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", inc,
            "-I", os.path.join(inc, "torch", "csrc", "api", "include"), "-I", sysconfig.get_paths()["include"],
            "-o", out, SRC_MARSHAL, "-L", lib, "-ltorch_python", "-ltorch_cpu", "-lc10", f"-Wl,-rpath,{lib}"]


def lib_path(variant: str = "bf16") -> str:
    return os.path.join(PKG, LIBS[variant])


def build_all(verbose: bool = False) -> list[str]:
    """Compile both variants and the marshalling module (in parallel); raises on any compiler error."""
    procs = []
    jobs = [(os.path.join(PKG, name), lambda tmp, v=variant: command(v, tmp)) for variant, name in LIBS.items()]
    jobs.append((MARSHAL, marshal_command))
    for out, make in jobs:
        tmp = out + ".tmp"
        cmd = make(tmp)
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((out, tmp, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    built = []
    errors = []
    for out, tmp, p in procs:
        log, _ = p.communicate()
        text = log.decode(errors="replace")
        # hipcc's host pass does not know the packed-fp32 feature and says so; harmless
        text = "\n".join(line for line in text.splitlines() if "packed-fp32-ops" not in line)
        if p.returncode != 0:
            errors.append(f"{os.path.basename(out)}:\n{text}")
            continue
        if verbose and text.strip():
            print(text)
        os.replace(tmp, out)
        built.append(out)
    if errors:
        raise RuntimeError("HIP build failed:\n" + "\n".join(errors))
    return built


def up_to_date(variant: str = "bf16") -> bool:
    """Whether the library variant and the marshalling module are no older than their sources."""
    return all(os.path.exists(out) and all(os.path.getmtime(d) <= os.path.getmtime(out) for d in deps)
               for out, deps in ((lib_path(variant), DEPS), (MARSHAL, [SRC_MARSHAL])))


if __name__ == "__main__":
    for path in build_all(verbose="-v" in sys.argv):
        print("built", path)
