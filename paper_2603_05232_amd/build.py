"""Builds libslidesparse.so (HIP kernels + C ABI, hipcc for gfx950) and the extension module _calls (host C++), in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libslidesparse.so")
CALLS = os.path.join(PKG, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ("lift_quant.hip", "prune_quant.hip", "decompose.hip", "gemm.hip", "gemm_skinny.hip", "gemm_mid.hip", "gemm_wide.hip", "gemm_slim.hip", "gemm_small.hip", "gemm_lifted.hip", "gemm_fused.hip", "gemm_fused_narrow.hip")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-inline-asm",      # the direct-to-LDS loads name M0 as clobbered, which clang reports as a reserved register
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("command failed: " + " ".join(cmd) + "\n" + out)
    return out


def _calls_command(obj: str):
    """Compiler command of the extension module (torch's headers; the torch libraries it needs are loaded by then)."""
    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    return [os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DSS_TORCH_VERSION="{torch.__version__}"', "-I" + os.path.join(ROOT, "include"), "-I" + inc,
            "-I" + os.path.join(inc, "torch", "csrc", "api", "include"), "-I/opt/rocm/include", "-I" + sysconfig.get_paths()["include"],
            "-c", os.path.join(CSRC, "py_calls.cpp"), "-o", obj]


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared library and the extension module; always recompiles."""
    import torch
    os.makedirs(OBJ, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = [os.path.join(OBJ, s.replace(".hip", ".o")) for s in SOURCES]
    calls_obj = os.path.join(OBJ, "py_calls.o")
    commands = [[hipcc, *FLAGS, "-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)] + [_calls_command(calls_obj)]
    with ThreadPoolExecutor(max_workers=len(commands)) as ex:
        outs = list(ex.map(_run, commands))
    outs.append(_run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]))
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    outs.append(_run([os.environ.get("CXX", "g++"), "-shared", "-o", CALLS, calls_obj, "-L" + torch_lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]))
    if verbose:
        print("\n".join(o for o in outs if o.strip()))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
