"""Builds the HIP library for gfx950 with hipcc (cross-compiles without a GPU) and the binding's native half."""
from __future__ import annotations

import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libmoe_rbf.so")
SOURCES = ["api.hip", "plan.hip", "dispatch.hip", "combine.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed-fp32 instruction selection is switched off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]
# The library depends on the HIP runtime by soname (libamdhip64.so.7).  A process that already holds a
# runtime with that soname (PyTorch ships its own copy) keeps using that one: the Python binding makes
# sure torch's copy is loaded first, so streams and device pointers belong to ONE runtime.


def build_library(out: str = LIB, defines: dict | None = None, verbose: bool = False,
                  extra_flags: list | None = None) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *(extra_flags or []), "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    for k, v in (defines or {}).items():
        cmd.append(f"-D{k}={v}")
    cmd += ["-o", out] + [os.path.join(CSRC, s) for s in SOURCES]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    log = "\n".join(l for l in (res.stdout + res.stderr).splitlines() if noise not in l and l.strip())
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed:\n{log}")
    if verbose and log:
        print(log)
    return out


def build_marshal(out: str = os.path.join(PKG, "_marshal.so")) -> str:
    """The binding's native argument marshalling (host code; reads torch tensors, so it is built against this torch).

    NDEBUG leaves out a thread-local counter of pybind11's headers.  A library with thread-local storage that is loaded late and
    never touches it makes every other library's thread-local accesses take the C library's slow path (glibc 2.35): torch's own
    calls were 10 to 20 % slower."""
    import sysconfig
    import torch
    from .binding import _interpreter
    at = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-DNDEBUG", "-Wall", "-I", os.path.join(ROOT, "include"),
           "-isystem", os.path.join(at, "include"), "-isystem", os.path.join(at, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DMOE_BUILT_FOR="{_interpreter(torch)}"',
           "-o", out, os.path.join(CSRC, "marshal.cpp"), "-L", os.path.join(at, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10",
           "-Wl,-rpath," + os.path.join(at, "lib")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"g++ failed:\n{res.stdout}{res.stderr}")
    return out


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_marshal())
