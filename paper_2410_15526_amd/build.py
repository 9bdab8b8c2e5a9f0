"""Compile the HIP library ``libsdp4.so`` for gfx950 with hipcc, in-tree.

Usable as ``python -m paper_2410_15526_amd.build``.  Each source compiles
to an object under ``_build/`` (in parallel), then one shared library is
linked next to this file.  Where a ROCm build of torch is installed, so is
``_binding.so``, the Python binding's argument marshalling (a CPython
extension on torch's headers); the library itself needs only hipcc.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libsdp4.so")
SOURCES = ["k_qwd.hip", "k_grad.hip", "k_sr.hip", "k_reduce.hip", "k_reduce_f32_in8.hip", "k_reduce_f32_in4.hip",
           "launch.cpp", "abi.cpp"]
BINDING = os.path.join(PKG, "_binding.so")
ARCH = "gfx950"

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                               # every fused multiply-add is written out
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", INCLUDE, "-I", CSRC,
]


def hipcc() -> str:
    p = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(p):
        raise RuntimeError("hipcc not found (ROCm is required to build the HIP library)")
    return p


def _compile(src: str, bdir: str, defines) -> str:
    obj = os.path.join(bdir, src + ".o")
    cmd = [hipcc(), *FLAGS, *[f"-D{d}" for d in defines], "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build_binding(out: str = BINDING) -> str | None:
    """Compile ``_binding.so`` with g++ (host code only); None, with nothing
    built, where there is no torch for it or torch is not a ROCm build."""
    import sysconfig

    try:
        import torch
    except ImportError:
        return None
    if torch.version.hip is None:
        return None
    troot = os.path.dirname(torch.__file__)
    tmp = out + f".tmp{os.getpid()}"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DSDP4_TORCH_VERSION="{torch.__version__}"', "-I", INCLUDE,
           "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(troot, "include"),
           "-isystem", os.path.join(troot, "include", "torch", "csrc", "api", "include"),
           "-isystem", os.path.join(os.path.dirname(os.path.dirname(hipcc())), "include"),
           os.path.join(CSRC, "binding.cpp"), "-o", tmp, "-L", os.path.join(troot, "lib"),
           "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for binding.cpp:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, out)
    return out


def build(verbose: bool = False, defines=(), out: str | None = None, build_dir: str | None = None) -> str:
    """Compile and link.  ``out`` and ``build_dir`` put the library (alone) and
    its objects somewhere else, ``defines`` are macros for hipcc: for builds of
    changed sources, since the committed ones read no macro."""
    bdir = build_dir or BUILD
    lib = out or LIB
    os.makedirs(bdir, exist_ok=True)
    with cf.ThreadPoolExecutor(len(SOURCES) + 1) as ex:
        binding = ex.submit(build_binding, BINDING) if out is None else None
        objs = list(ex.map(lambda s: _compile(s, bdir, defines), SOURCES))
    tmp = lib + f".tmp{os.getpid()}"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, lib)
    if binding is not None and binding.result() is None and verbose:
        print("no ROCm build of torch: _binding.so is left out")
    if verbose:
        print(f"built {lib}")
    return lib


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
