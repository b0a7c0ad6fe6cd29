"""Build libunstep.so (HIP kernels + C ABI host code) for gfx950, in-tree.

    python paper_2609_32518_amd/build.py [-v]

Run by path (not with -m): importing the package loads the library this script builds.

Every source under csrc/ is compiled by hipcc to an object under _build/ and the
objects are linked into paper_2609_32518_amd/libunstep.so, with ROCm's rocSOLVER and
rocBLAS (the init-time SVD).  Device code is built
with packed-fp32 instructions disabled.  native/calls.cpp, the binding's native calls, becomes
paper_2609_32518_amd/_calls.so, a CPython extension module linked to torch and to libunstep.so.
"""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libunstep.so")
CALLS_SRC = os.path.join(PKG, "native", "calls.cpp")
CALLS = os.path.join(PKG, "_calls.so")

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
ARCH = "gfx950"
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", f"-I{INCLUDE}", f"-I{CSRC}"]
DEVICE = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libunstep.so)")


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".cpp", ".hip")))


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [hipcc()] + COMMON + DEVICE + ["-c", src, "-o", obj]
    if src.endswith(".cpp"):
        cmd = [hipcc()] + COMMON + ["-x", "c++", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", "-c", src,
                                  "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compiling {src} failed:\n{r.stdout}\n{r.stderr}")
    # show warnings other than hipcc's note that the host pass ignores the device feature flag
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if warn and verbose:
        print(warn, file=sys.stderr)
    return obj


def _run(cmd, what: str, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{r.stdout}\n{r.stderr}")


def _torch_dir() -> str:
    import importlib.util
    return os.path.dirname(importlib.util.find_spec("torch").origin)


def _compile_calls(verbose: bool) -> str:
    """The object of native/calls.cpp (host code only, against torch's headers)."""
    cxx = os.environ.get("CXX") or shutil.which("g++") or shutil.which("c++")
    if not cxx:
        raise RuntimeError("no C++ compiler found")
    inc = os.path.join(_torch_dir(), "include")
    obj = os.path.join(BUILD, "calls.cpp.o")
    _run([cxx, "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", f"-I{INCLUDE}", f"-isystem{inc}",
          f"-isystem{inc}/torch/csrc/api/include", f"-isystem{ROCM}/include",
          f"-isystem{sysconfig.get_paths()['include']}", "-c", CALLS_SRC, "-o", obj], f"compiling {CALLS_SRC}", verbose)
    return obj


def _link_calls(obj: str, verbose: bool) -> None:
    cxx = os.environ.get("CXX") or shutil.which("g++") or shutil.which("c++")
    tl = os.path.join(_torch_dir(), "lib")
    tmp = CALLS + ".tmp"
    _run([cxx, "-shared", "-o", tmp, obj, f"-L{PKG}", "-lunstep", f"-L{tl}", "-ltorch_python", "-ltorch", "-ltorch_cpu",
          "-lc10", "-lc10_hip", "-Wl,-z,now", "-Wl,-rpath,$ORIGIN", f"-Wl,-rpath,{tl}"], "linking _calls.so", verbose)
    os.replace(tmp, CALLS)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        calls = ex.submit(_compile_calls, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
        calls_obj = calls.result()
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs + [
        f"-L{ROCM}/lib", "-lrocsolver", "-lrocblas", f"-Wl,-rpath,{ROCM}/lib"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"linking libunstep.so failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    _link_calls(calls_obj, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
