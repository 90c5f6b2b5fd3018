"""Build the gfx950 HIP library ``libobjectcache.so`` in-tree with hipcc."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libobjectcache.so")
# the Python binding's argument marshalling (a CPython module, host code only)
MARSHAL_SRC = os.path.join(PKG, "native", "marshal.cpp")
MARSHAL = os.path.join(PKG, "_marshal.so")
BUILD_DIR = os.path.join(ROOT, "_build")
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-I", INCLUDE, "-I", CSRC,
    # packed fp32 VALU ops stay disabled on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


# Host code instrumented with AddressSanitizer (device code as usual): a
# separate library under _build/asan for sanitizer runs of the host paths
ASAN_DIR = os.path.join(BUILD_DIR, "asan")
ASAN_LIB = os.path.join(ASAN_DIR, "libobjectcache.so")
ASAN_FLAGS = ["-O1", "-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fno-omit-frame-pointer"]


def _compile(src: str, asan: bool = False) -> str:
    obj = os.path.join(ASAN_DIR if asan else BUILD_DIR, os.path.basename(src) + ".o")
    flags = [f for f in COMMON if f != "-O3"] + ASAN_FLAGS if asan else COMMON
    cmd = [HIPCC, *flags, "-c", src, "-o", obj]
    if src.endswith(".cpp"):
        cmd[1:1] = ["-x", "hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def _build_marshal() -> None:
    tmp = MARSHAL + ".tmp"
    r = subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I", INCLUDE,
                        "-I", sysconfig.get_paths()["include"], MARSHAL_SRC, "-o", tmp], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compiling {MARSHAL_SRC} failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, MARSHAL)


def build(verbose: bool = False, asan: bool = False) -> str:
    """Compile every source for gfx950 and link the library in-tree (with
    asan, the sanitizer build of the host code at ASAN_LIB instead)."""
    out = ASAN_LIB if asan else LIB
    os.makedirs(os.path.dirname(out) if asan else BUILD_DIR, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda f: _compile(f, asan), srcs))
    tmp = out + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp,
           "-lpthread", "-lrocblas", "-lrocprofiler-sdk-roctx"]
    if asan:
        cmd += ["-Xarch_host", "-fsanitize=address", "-shared-libsan"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, out)
    _build_marshal()
    if verbose:
        print(f"built {out}")
    return out


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
