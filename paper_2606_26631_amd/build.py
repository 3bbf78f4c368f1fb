"""Build the HIP library libprcr.so for gfx950 (in-tree, next to this file).

Every source is compiled with hipcc for gfx950 only; the library is linked into
the package directory so that the Python binding, the tests and the benchmark
load it from the source tree.  The binding's native module (host code, against the
installed torch and Python) is built beside it.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OUT = os.path.join(PKG, "libprcr.so")
BUILD_DIR = os.path.join(ROOT, "_build")

# The bandwidth measurement's reference copies (a plain streaming copy and a copy
# with the rebinding kernel's access pattern), in a library of their own: they are
# not part of the PRCR path or its ABI.
COPYREF_SOURCES = ["copyref.hip"]
COPYREF_OUT = os.path.join(PKG, "libprcr_copyref.so")
SOURCES = ["api.cpp", "axis_map.cpp", "decode.hip", "decode_static.hip", "prefill.hip", "reassign.hip", "rebind.hip", "store_raw.hip"]

# The binding's native module: C++ against torch's and Python's headers.
NATIVE_SOURCE = "native_calls.cpp"
NATIVE_OUT = os.path.join(PKG, "_prcr_native.so")

# Packed-FP32 instructions are disabled for all device code; the host pass of
# hipcc warns that it does not know the feature, which is harmless.
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         f"-I{INCLUDE}", f"-I{CSRC}"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; install ROCm or set HIPCC")


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"]
    cmd = [hipcc(), *lang, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr, file=sys.stderr)
    return obj


def _link(objs, out: str, verbose: bool) -> None:
    tmp = out + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, out)


def _cxx() -> str:
    return os.environ.get("CXX", "g++")


def _native_lacks() -> str:
    """What the native module's build does not find here ("" if nothing)."""
    try:
        import torch.utils.cpp_extension  # noqa: F401
    except ImportError as e:
        return f"torch ({e})"
    if shutil.which(_cxx()) is None:
        return f"a host compiler ({_cxx()})"
    if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        return "Python's headers"
    return ""


def _compile_native(verbose: bool) -> str:
    import torch
    from torch.utils.cpp_extension import include_paths
    obj = os.path.join(BUILD_DIR, os.path.splitext(NATIVE_SOURCE)[0] + ".o")
    rocm = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc()))), "include")
    incs = [*include_paths(), sysconfig.get_paths()["include"], rocm]
    cmd = [_cxx(), "-O2", "-std=c++17", "-fPIC", "-Wall", "-fvisibility=hidden",
           "-D__HIP_PLATFORM_AMD__", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           '-DPRCR_BUILT_FOR="torch {}, Python {}.{}"'.format(torch.__version__, *sys.version_info[:2]),
           f"-I{INCLUDE}", *[a for i in incs for a in ("-isystem", i)],
           "-c", os.path.join(CSRC, NATIVE_SOURCE), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"the host compiler failed for {NATIVE_SOURCE}:\n{r.stdout}\n{r.stderr}")
    return obj


def _link_native(obj: str, verbose: bool) -> None:
    from torch.utils.cpp_extension import library_paths
    tmp = NATIVE_OUT + ".tmp"
    cmd = [_cxx(), "-shared", obj, "-o", tmp, *[f"-L{d}" for d in library_paths()],
           "-ltorch_python", "-ltorch_cpu", "-lc10", f"-L{PKG}", f"-l:{os.path.basename(OUT)}",
           "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, NATIVE_OUT)


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link libprcr.so, the measurement's reference
    copy kernels into libprcr_copyref.so, and the binding's native module; returns
    libprcr.so's path.  The native module is left out, with a line on stderr, where torch, a
    host compiler or Python's headers are missing: a C program needs only the library, and
    the binding makes its calls without the module."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    lacks = _native_lacks()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + len(COPYREF_SOURCES) + 1)) as ex:
        native = None if lacks else ex.submit(_compile_native, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES + COPYREF_SOURCES))
    _link(objs[:len(SOURCES)], OUT, verbose)
    _link(objs[len(SOURCES):], COPYREF_OUT, verbose)
    made = False
    try:
        if native is None:
            print(f"the binding's native module is not built: {lacks} is missing", file=sys.stderr)
        else:
            _link_native(native.result(), verbose)
            made = True
    finally:
        if not made and os.path.exists(NATIVE_OUT):
            os.remove(NATIVE_OUT)     # no earlier build's module beside a new library
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
