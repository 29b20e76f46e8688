"""Builds libdfsattn.so (HIP kernels + C ABI) for gfx950 and, for the running Python and torch, the module _calls (csrc/calls.cpp) with
hipcc, in-tree."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdfsattn.so")
SOURCES = ["api.hip", "hilbert.hip", "permute.hip", "score.hip", "select.hip", "attn.hip", "recall.hip", "probe.hip", "small.hip"]
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))      # another Python does not take it for its own
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ROCM = os.path.dirname(os.path.dirname(HIPCC)) if os.path.isabs(HIPCC) else "/opt/rocm"
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _calls_command() -> list[str] | None:
    """None where the headers of Python or of a torch for ROCm are missing: the binding then does these calls in Python."""
    try:
        import torch
        from torch.utils import cpp_extension
        include = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"], os.path.join(ROCM, "include")]
    except (ImportError, OSError):
        return None
    for header in ("Python.h", "torch/csrc/autograd/python_variable.h", "c10/hip/HIPStream.h"):
        if not any(os.path.exists(os.path.join(d, header)) for d in include):
            return None
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return [HIPCC, "-no-hip-rt", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", f'-DDFS_TORCH_VERSION="{torch.__version__}"',
            *(x for d in include for x in ("-isystem", d)), "-x", "c++", os.path.join(CSRC, "calls.cpp"), "-o", CALLS,
            f"-L{HERE}", "-l:" + os.path.basename(LIB), f"-L{lib}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]


def build_library(verbose: bool = False, jobs: int = 6) -> str:
    """Compiles every translation unit and links the shared library and the module of its calls; returns the library's path."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if len(procs) >= jobs:
            _wait(procs.pop(0), verbose)
    for p in procs:
        _wait(p, verbose)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    out = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if out.returncode != 0:
        raise RuntimeError("link failed:\n" + out.stdout)
    for old in glob.glob(os.path.join(HERE, "_calls*.so")):      # whatever Python they are for, they call the library as it was
        os.remove(old)
    calls = _calls_command()
    if calls:
        _wait(("calls.cpp", subprocess.Popen(calls, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)), verbose)
    return LIB


def _wait(item, verbose):
    src, proc = item
    out, _ = proc.communicate()
    # the host pass does not know the device-only target feature and says so; that is harmless
    lines = [l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip()]
    if proc.returncode != 0:
        raise RuntimeError(f"compilation failed on {src}:\n" + "\n".join(lines))
    if verbose and lines:
        print("\n".join(lines), flush=True)


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
