"""Build libfasgd.so (HIP, gfx950) with hipcc and the binding's _marshal.so (host C++ against torch's headers) with
g++, both in-tree."""
import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libfasgd.so")
SOURCES = ["fasgd_api.hip", "dense.hip", "bfasgd.hip", "segments.hip", "pushes.hip", "selfcheck.hip", "anchor.hip"]

MARSHAL = os.path.join(PKG, "_marshal.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Werror",
    "-I", os.path.join(ROOT, "include"),
    # packed fp32 instructions stay off: hand-written or compiler-generated,
    # v_pk_{add,mul,fma}_f32 are not used by this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the host pass does not know the feature above
    "-Wno-unknown-warning-option",
]


def build(verbose: bool = False, extra_flags=()) -> str:
    if shutil.which(HIPCC) is None and not os.path.exists(HIPCC):
        raise RuntimeError(f"hipcc not found at {HIPCC}")
    os.makedirs(BUILD, exist_ok=True)
    objs = []
    for src in SOURCES:
        obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
        cmd = [HIPCC, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    build_marshal(verbose)
    return LIB


def build_marshal(verbose: bool = False):
    """The native argument marshalling of the binding (csrc/marshal.cpp).  The library does not need it: without a
    host compiler, Python's headers or torch it is left out, and the binding marshals in Python."""
    cxx = os.environ.get("CXX", "g++")
    try:
        import torch
        from torch.utils import cpp_extension
    except ImportError:
        torch = None
    if torch is None or not shutil.which(cxx) or not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        print(f"{os.path.basename(MARSHAL)} left out: it needs {cxx}, Python.h and torch", file=sys.stderr, flush=True)
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)      # an older build's
        return None
    inc = [f"-I{d}" for d in (os.path.join(ROOT, "include"), *cpp_extension.include_paths(),
                              sysconfig.get_paths()["include"], "/opt/rocm/include")]
    tmp = MARSHAL + ".tmp"
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DFASGD_TORCH_VERSION="{torch.__version__}"', *inc,
           os.path.join(CSRC, "marshal.cpp"), "-o", tmp, *[f"-L{d}" for d in cpp_extension.library_paths()],
           "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, MARSHAL)
    return MARSHAL


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
