"""Build libmacko.so (host C++ + gfx950 HIP kernels) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmacko.so")
BINDING = os.path.join(HERE, "_native" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["macko_host.cpp", "macko_spmv.hip", "macko_gemv.hip", "macko_encode_gpu.hip", "macko_spmm.hip", "macko_spmm_tile.hip", "macko_decode_gpu.hip"]
HEADERS = ["macko_internal.h", "macko_device.h", "macko_plan.h", "macko_decode.h"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    # keep the compiler from forming packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # leading scalar kernel arguments arrive in registers instead of through a load
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-function",
]


def library_path() -> str:
    return LIB


def _older(built: str, sources) -> bool:
    deps = [os.path.join(CSRC, f) for f in sources] + [os.path.join(ROOT, "include", "macko.h")]
    return not os.path.exists(built) or any(os.path.getmtime(d) > os.path.getmtime(built) for d in deps)


def is_stale() -> bool:
    return _older(LIB, SOURCES + HEADERS)


def binding_is_stale() -> bool:
    """The native part of the Python binding is missing, or older than its sources or the PyTorch it was built against."""
    import torch
    return _older(BINDING, ["binding_torch.cpp"]) or os.path.getmtime(torch.version.__file__) > os.path.getmtime(BINDING)


def build_library(force: bool = True, verbose: bool = False, extra_flags=()) -> str:
    """Compile every source for gfx950 and link the shared library, and the native part of the binding if it is stale."""
    try:
        if binding_is_stale():
            build_binding(verbose)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:     # no PyTorch, no headers: the binding goes through ctypes
        print(f"the native part of the binding is not built: {e}", file=sys.stderr)
    if not force and not is_stale():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + f".tmp{os.getpid()}"
    cmd = [hipcc, *HIPCC_FLAGS, *extra_flags, "-shared", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           "-x", "hip", *[os.path.join(CSRC, s) for s in SOURCES], "-o", tmp, "-lpthread"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


def build_binding(verbose: bool = False) -> str:
    """Compile the native part of the Python binding (host code only) against the installed PyTorch."""
    import torch
    base = os.path.dirname(torch.__file__)
    inc = os.path.join(base, "include")
    tmp = BINDING + f".tmp{os.getpid()}"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-w",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(ROOT, "include"), "-I", inc, "-I", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-I", sysconfig.get_paths()["include"], "-I", "/opt/rocm/include", os.path.join(CSRC, "binding_torch.cpp"), "-o", tmp,
           "-L", os.path.join(base, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python",
           "-Wl,-rpath," + os.path.join(base, "lib")]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, BINDING)
    return BINDING


if __name__ == "__main__":
    build_binding(verbose=True)
    print(build_library(verbose=True, extra_flags=sys.argv[1:]))
    print(BINDING)
