"""Build libhydra.so (HIP kernels for gfx950 + the C ABI) in-tree with hipcc, and _hydra_native.so (the Python
binding's call path, host code against torch's headers) with g++.

Usage:  python -m paper_2309_00754_amd.build [--verbose]
Objects go to ``_build/`` at the repository root; the shared libraries are
written next to this file.  Every call recompiles.  libhydra.so does not wait
for _hydra_native.so: without the latter (no torch headers, another ABI) the
binding's calls go through ctypes.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import shutil
import subprocess
import sys
import warnings

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libhydra.so")
NATIVE_SRC = os.path.join(PKG, "native", "binding.cpp")
NATIVE = os.path.join(PKG, "_hydra_native.so")
ARCH = "gfx950"

# Packed fp32 instructions are disabled for device code (the host pass warns
# that it does not know the feature; that warning is harmless).
DEVICE_FLAGS = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
COMMON = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-I", INCLUDE, "-I", CSRC, "-Wall"]


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP library cannot be built")


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [_hipcc(), *COMMON, *DEVICE_FLAGS, "-c", src, "-o", obj]
    if src.endswith(".cpp"):
        cmd = [_hipcc(), *COMMON, "-x", "hip", *DEVICE_FLAGS, "-c", src, "-o", obj]
    if verbose:
        cmd.insert(1, "-Rpass-analysis=kernel-resource-usage")
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    msg = "\n".join(l for l in (res.stdout + res.stderr).splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{msg}")
    if verbose and msg.strip():
        print(msg)
    return obj


def _run(cmd, what: str) -> None:
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{what} failed:\n" + res.stdout + res.stderr)


def _compile_native() -> str:
    import sysconfig

    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    obj = os.path.join(BUILD, "binding.o")
    _run([shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem", inc,
          "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
          "-isystem", sysconfig.get_paths()["include"], "-c", NATIVE_SRC, "-o", obj], "g++ on the native binding")
    return obj


def _link_native(obj: str) -> None:
    """Against the libhydra.so beside it; torch's libraries are those of the running process."""
    import torch
    tmp = NATIVE + ".tmp"
    _run([shutil.which("g++") or "g++", "-shared", obj, "-o", tmp, "-L", PKG, "-l:libhydra.so", "-Wl,-rpath,$ORIGIN",
          "-L", os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10",
          "-lc10_hip"], "link of the native binding")
    os.replace(tmp, NATIVE)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        native = ex.submit(_compile_native)
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    tmp = LIB + ".tmp"
    _run([_hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-Wl,-soname,libhydra.so", *objs, "-o", tmp], "link")
    os.replace(tmp, LIB)
    try:
        _link_native(native.result())
    except Exception as e:  # noqa: BLE001 (whatever it was, libhydra.so is there)
        if os.path.exists(NATIVE):
            os.remove(NATIVE)  # (of an earlier build: not to be loaded with this libhydra.so)
        warnings.warn(f"_hydra_native.so is not built, calls go through ctypes: {e}", RuntimeWarning, stacklevel=2)
    return LIB


if __name__ == "__main__":
    print(build(verbose="--verbose" in sys.argv))
