"""Build libsrft_kv.so (the product) and libsrft_measure.so (measurement aids) in-tree with hipcc, for gfx950, and the
binding's native marshalling (_marshal, a CPython extension, host code) with g++.

Every translation unit under csrc/ is compiled to an object of its own (in parallel), then linked; objects whose
source and headers are older than they are are reused unless ``force`` is set.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import shutil
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libsrft_kv.so")
LIB_MEASURE = os.path.join(PKG, "libsrft_measure.so")
SRC_MARSHAL = os.path.join(CSRC, "host", "marshal.cpp")
LIB_MARSHAL = os.path.join(PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))      # (of this interpreter, and found by no other)
SRC = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "kernels", "*.hip")))
SRC_MEASURE = sorted(glob.glob(os.path.join(CSRC, "measure", "*.hip")))
HEADERS = sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h")))
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU forms are kept out of the generated code on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA accumulators in ordinary VGPRs: the vector-ALU tail reads them without v_accvgpr_read copies
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    # the first arguments of a kernel arrive in scalar registers instead of being fetched at its start (0.2-0.3 us of a small launch)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-I", os.path.join(ROOT, "include"),
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def _run(cmd: list[str], verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + res.stdout + res.stderr)


def _object(src: str, force: bool, verbose: bool, extra: list[str]) -> str:
    obj = os.path.join(OBJ, os.path.relpath(src, CSRC).replace(os.sep, "_") + ".o")
    newest = max(os.path.getmtime(f) for f in [src, *HEADERS, os.path.abspath(__file__)])
    if force or not os.path.exists(obj) or os.path.getmtime(obj) < newest:
        _run([hipcc(), *FLAGS, *extra, "-c", src, "-o", obj], verbose)
    return obj


def _marshal_command(include: str = os.path.join(ROOT, "include")) -> list[str]:
    import torch
    at = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc())))
    return [shutil.which("g++") or "c++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem", sysconfig.get_paths()["include"],
            "-isystem", os.path.join(at, "include"), "-isystem", os.path.join(at, "include", "torch", "csrc", "api", "include"),
            "-isystem", os.path.join(rocm, "include"), "-I", include, SRC_MARSHAL, "-L", os.path.join(at, "lib"),
            "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def _marshal_lacks() -> str:
    """What the extension needs and is not there ("": nothing)."""
    try:
        import torch
    except ImportError:
        return "torch"
    headers = [os.path.join(sysconfig.get_paths()["include"], "Python.h"),
               os.path.join(os.path.dirname(torch.__file__), "include", "torch", "csrc", "autograd", "python_variable.h")]
    missing = [] if shutil.which("g++") or shutil.which("c++") else ["g++"]
    return ", ".join(missing + [h for h in headers if not os.path.exists(h)])


def _marshal(force: bool, verbose: bool) -> None:
    """The CPython extension that binding.py calls: torch's headers, no HIP code.  Where a compiler or headers for it are missing the
    libraries are built all the same, and the binding makes every call through ctypes."""
    if lacks := _marshal_lacks():
        print(f"_marshal is not built, calls go through ctypes: no {lacks}", flush=True)
        if os.path.exists(LIB_MARSHAL):
            os.remove(LIB_MARSHAL)                             # (one of other sources)
        return
    newest = max(os.path.getmtime(f) for f in (SRC_MARSHAL, *HEADERS, os.path.abspath(__file__)))
    if os.path.exists(untagged := os.path.join(PKG, "_marshal.so")):       # (from builds that named it so: any interpreter would load it)
        os.remove(untagged)
    if force or not os.path.exists(LIB_MARSHAL) or os.path.getmtime(LIB_MARSHAL) < newest:
        _run([*_marshal_command(), "-shared", "-o", LIB_MARSHAL], verbose)


def build(verbose: bool = False, extra: list[str] | None = None, force: bool = True, jobs: int | None = None) -> str:
    """Compile and link the libraries and the extension; returns the path of libsrft_kv.so."""
    os.makedirs(OBJ, exist_ok=True)
    extra = list(extra or [])
    jobs = jobs or min(8, os.cpu_count() or 1)
    with cf.ThreadPoolExecutor(max_workers=jobs) as pool:
        marshal = pool.submit(_marshal, force, verbose)
        objs = list(pool.map(lambda s: _object(s, force, verbose, extra), SRC + SRC_MEASURE))
        marshal.result()
    n = len(SRC)
    _run([hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs[:n], "-o", LIB], verbose)
    _run([hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs[n:], "-o", LIB_MEASURE], verbose)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(verbose=True, force="--incremental" not in sys.argv))
