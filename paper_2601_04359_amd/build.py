"""Builds libpackcache.so (gfx950) in-tree with hipcc, and the compiled half of the binding with g++.
`python -m paper_2601_04359_amd.build`"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB_DIR = os.path.join(PKG, "lib")
LIB_PATH = os.path.join(LIB_DIR, "libpackcache.so")
MARSHAL_PATH = os.path.join(PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["host.cpp", "rope.hip", "attn.hip", "score.hip", "compact.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _run(cmd):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode != 0:
        raise RuntimeError("command failed: " + " ".join(cmd) + "\n" + out)
    return out


def build_marshal() -> str:
    """The compiled half of the binding: host code against Python's and torch's headers.  NDEBUG keeps it free
    of thread-local storage (pybind11's reference counter): loading a module that has some and never touches
    it leaves every later thread-local access of the process on the loader's slow path (each torch call
    4.4 -> 4.75 us)."""
    for old in glob.glob(os.path.join(os.path.dirname(MARSHAL_PATH), "_marshal*.so")):
        os.remove(old)    # none at all rather than one of an older build
    import torch
    at = os.path.dirname(torch.__file__)
    lib = os.path.join(at, "lib")
    return _run(["g++", "-O2", "-DNDEBUG", "-std=c++17", "-fPIC", "-shared", "-I" + os.path.join(ROOT, "include"),
                 "-I" + os.path.join(at, "include"), "-I" + os.path.join(at, "include", "torch", "csrc", "api", "include"),
                 "-I" + sysconfig.get_paths()["include"], f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                 f'-DPC_TORCH_VERSION="{torch.__version__}"',
                 os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL_PATH,
                 "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10", "-Wl,-rpath," + lib])


def build_library(verbose: bool = False) -> str:
    """Compile every translation unit and link the shared library; always recompiles.  The binding's compiled
    half is built where it can be: the library does not need it."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    obj_dir = os.path.join(PKG, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    os.makedirs(LIB_DIR, exist_ok=True)
    objs = [os.path.join(obj_dir, os.path.splitext(s)[0] + ".o") for s in SOURCES]

    def one(pair):
        src, obj = pair
        return _run([hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj])

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        logs = list(ex.map(one, zip(SOURCES, objs)))
    logs.append(_run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB_PATH]))
    try:
        logs.append(build_marshal())
    except (ImportError, OSError, RuntimeError) as e:   # no torch, no g++, no headers
        warnings.warn(f"the binding's compiled half was not built, calls go through ctypes: {e}")
    if verbose:
        print("\n".join(l for l in logs if l))
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
    sys.exit(0)
