"""Builds libvidiq.so (the C-ABI library with the gfx950 kernels) in-tree with hipcc, and the torch extension.

Usage: python -m paper_2406_02540_amd.build
"""
from __future__ import annotations

import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libvidiq.so")
CEILINGS_PATH = os.path.join(PKG_DIR, "vq_ceilings")  # stand-alone program, see csrc/vq_ceilings.hip
SOURCES = ["vq_api.hip", "vq_quantize.hip", "vq_fused.hip", "vq_fused_gelu.hip", "vq_gemm.hip", "vq_gemm_192.hip", "vq_gemm_192w4.hip", "vq_gemm_tiles.hip", "vq_gemm_split.hip",
           "vq_linear_small.hip"]

EXT_PATH = os.path.join(PKG_DIR, "_vq_torch.so")  # the torch side (csrc/vq_torch.cpp): host code only

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-ffp-contract=off",          # every fp32 operation rounds on its own
    "-fno-fast-math",
    # packed-fp32 instructions are not used in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def cxx() -> str:
    """The C++ compiler of the torch extension: $CXX, g++, or the clang++ that hipcc drives."""
    clang = os.path.join(os.path.dirname(os.path.realpath(shutil.which(hipcc()) or hipcc())), "amdclang++")
    for cand in (os.environ.get("CXX"), "g++", clang):
        if cand and shutil.which(cand.split()[0]):
            return cand
    return "c++"


def ext_command(out: str) -> list:
    """The compiler call for the torch extension (plain C++ against torch's headers)."""
    import torch
    root = os.path.dirname(torch.__file__)
    return [*cxx().split(), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-I", os.path.join(ROOT, "include"), "-I", os.path.join(root, "include"),
            "-I", os.path.join(root, "include", "torch", "csrc", "api", "include"), "-I", "/opt/rocm/include",
            "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "vq_torch.cpp"),
            "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-o", out]


def build(verbose: bool = True) -> str:
    """Compiles every source for gfx950 and links the shared library, then the torch extension. Always recompiles.

    The library needs hipcc only: without torch it is built alone, and it is in place before the extension is.
    """
    objs = []
    procs = []
    ext = None
    if importlib.util.find_spec("torch") is None:
        print("torch is not installed: libvidiq.so is built without its Python binding", flush=True)
    else:
        ext_tmp = EXT_PATH + ".tmp.%d" % os.getpid()
        cmd = ext_command(ext_tmp)
        if verbose:
            print(" ".join(cmd), flush=True)
        ext = subprocess.Popen(cmd)
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [hipcc(), *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
               "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd)))
        objs.append(obj)
    for src, p in procs:
        if p.wait() != 0:
            raise RuntimeError(f"hipcc failed on {src}")
    tmp = LIB_PATH + ".tmp.%d" % os.getpid()
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB_PATH)
    if ext is not None:
        if ext.wait() != 0:
            raise RuntimeError(f"{cxx()} failed on vq_torch.cpp")
        os.replace(ext_tmp, EXT_PATH)
    # the ceilings probe (register-only MFMA loop, copy kernel): its own small executable
    tmp = CEILINGS_PATH + ".tmp.%d" % os.getpid()
    cmd = [hipcc(), *[f for f in HIPCC_FLAGS if f != "-fPIC"], os.path.join(CSRC, "vq_ceilings.hip"), "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, CEILINGS_PATH)
    return LIB_PATH


if __name__ == "__main__":
    build()
    print("built", LIB_PATH)
    sys.exit(0)
