"""Builds libtf_gfx950.so (HIP kernels + C boundary) in-tree with hipcc.

hipcc cross-compiles for gfx950 without a GPU, so this runs anywhere the ROCm toolchain is
installed.  ``python -m paper_2512_09196_amd.build`` rebuilds unconditionally.
"""
from __future__ import annotations

import importlib.machinery
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libtf_gfx950.so")
PYCALL = os.path.join(HERE, "_tfcall" + importlib.machinery.EXTENSION_SUFFIXES[0])   # extension module of this interpreter, host code only
SOURCES = ["tf_gemm_lds.hip", "tf_gemm_lds_ragged.hip", "tf_gemm_lds_192.hip", "tf_gemm_lds_64x128.hip", "tf_gemm_stream.hip", "tf_gemm_any.hip", "tf_gemm_kshare.hip", "tf_vecmat.hip", "tf_sin.hip", "tf_gemm_simple.hip", "tf_api.hip", "tf_loop.cpp"]
HEADERS = ["tf_gemm_lds.h", "tf_internal.h", "tf_device.h", "tf_loop.h"]

# -packed-fp32-ops off: hipcc must not form v_pk_*_f32 from scalar float code on this target.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I" + os.path.join(ROOT, "include"),
         "-I" + CSRC, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def _newest_input() -> float:
    paths = [os.path.join(CSRC, f) for f in SOURCES + HEADERS + ["tf_pycall.cpp"]] + [os.path.join(ROOT, "include", "tf.h"), __file__]
    return max(os.path.getmtime(p) for p in paths)


def up_to_date() -> bool:
    wanted = (LIB,) if pycall_tools() is None else (LIB, PYCALL)
    return all(os.path.exists(f) and os.path.getmtime(f) >= _newest_input() for f in wanted)


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src + ".o")
    cmd = [_hipcc()] + FLAGS + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj


def pycall_tools():
    """(C++ compiler, folder of Python.h), or None where one of them is missing. (Not hipcc: it links the HIP runtime.)"""
    include = sysconfig.get_paths()["include"]
    cxx = shutil.which("g++") or shutil.which("c++") or shutil.which("clang++")
    return (cxx, include) if cxx and os.path.exists(os.path.join(include, "Python.h")) else None


def build_pycall():
    """Compile the extension module behind Problem.run for this interpreter. Returns its path, or None without the tools:
    Problem.run then calls the library through ctypes."""
    tools = pycall_tools()
    if tools is None:
        sys.stderr.write("no C++ compiler or no Python.h: %s is left out\n" % os.path.basename(PYCALL))
        return None
    tmp = PYCALL + ".tmp.%d" % os.getpid()
    cmd = [tools[0], "-O2", "-std=c++17", "-fPIC", "-shared", "-I" + tools[1], os.path.join(CSRC, "tf_pycall.cpp"), "-o", tmp]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("%s failed on tf_pycall.cpp:\n%s" % (tools[0], r.stdout))
    os.replace(tmp, PYCALL)
    return PYCALL


def build_library(force: bool = True) -> str:
    """Compile every source for gfx950 and link the shared library. Returns its path."""
    if not force and up_to_date():
        return LIB
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        pycall = ex.submit(build_pycall)
        objs = list(ex.map(_compile, SOURCES))
        pycall.result()
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(True))
