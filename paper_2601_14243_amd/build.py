"""Build libjet.so (the C-ABI HIP library) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libjet.so")
PROBE_LIB = os.path.join(HERE, "libjet_probe.so")     # measurement aid of bench.py, not part of the product ABI
HOST_LIB = os.path.join(HERE, "_jet_host.so")         # native marshalling of the tensor helpers (host code only)
SOURCES = ["jet_api.hip", "jet_quant.hip", "jet_fused.hip", "jet_gemm.hip"]
PROBE_SOURCES = ["jet_probe.hip"]
HEADERS = ["jet_internal.h", "jet_numerics.h", "jet_plan.h", "jet_tile_quant.h", os.path.join("..", "..", "include", "jet.h")]

# No fast-math: divisions, products and fmas must be the IEEE binary32 operations.
# Packed-fp32 instructions are switched off for the device compiler.
# Only the extern "C" entry points marked JET_API are exported.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(lib: str, sources, force: bool) -> None:
    srcs = [os.path.join(CSRC, s) for s in sources]
    if not force and os.path.exists(lib):
        newest = max(os.path.getmtime(p) for p in srcs + [os.path.join(CSRC, h) for h in HEADERS])
        if os.path.getmtime(lib) >= newest:
            return
    res = subprocess.run(["hipcc", *FLAGS, "-o", lib, *srcs], capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)


def _compile_host(force: bool) -> None:
    """The Python extension behind binding.py's tensor helpers: g++ against torch's headers, linked to libjet.so beside it."""
    src = os.path.join(CSRC, "jet_host.cpp")
    if not force and os.path.exists(HOST_LIB):
        if os.path.getmtime(HOST_LIB) >= max(os.path.getmtime(p) for p in (src, os.path.join(CSRC, HEADERS[-1]))):
            return
    import torch
    from torch.utils import cpp_extension
    rocm = cpp_extension.ROCM_HOME or "/opt/rocm"
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wno-unused-variable",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[f"-isystem{p}" for p in cpp_extension.include_paths()], f"-isystem{os.path.join(rocm, 'include')}",
           f"-isystem{sysconfig.get_paths()['include']}", "-o", HOST_LIB, src,
           f"-L{torch_lib}", "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", f"-L{HERE}", "-l:libjet.so",
           "-Wl,-rpath,$ORIGIN"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stdout + res.stderr)


def build(force: bool = True) -> str:
    """Compile every source: libjet.so (the product), libjet_probe.so (the benchmark's matrix-core rate probe) and the
    Python extension, without which the helpers work too.  Returns the path of libjet.so."""
    _compile(LIB, SOURCES, force)
    _compile(PROBE_LIB, PROBE_SOURCES, force)
    try:
        _compile_host(force)
    except (RuntimeError, OSError) as e:     # no g++, no headers, another torch: the library works without it
        if os.path.exists(HOST_LIB):
            os.remove(HOST_LIB)              # not one that is older than its source
        warnings.warn(f"the native marshalling was not built, binding.py stands in for it: {e}", RuntimeWarning)
    return LIB


if __name__ == "__main__":
    print(build())
