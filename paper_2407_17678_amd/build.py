"""Builds libs2attn.so (HIP kernels + C ABI) for gfx950 with hipcc, and _marshal.so (the Python side of its compute
calls) with the host compiler, in-tree.

Run as ``python -m paper_2407_17678_amd.build``.  hipcc cross-compiles without a GPU.
"""

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libs2attn.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["api.hip", "layout.cpp", "fwd_pipe_kernel.hip", "fwd_gather_kernel.hip", "bwd_kernel.hip", "bwd_merged_kernel.hip", "dq_pipe_kernel.hip", "dq_gemm_kernel.hip", "decode_kernel.hip", "probe_kernel.hip"]

COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function"]
# gfx950 only.  Packed-fp32 VALU forms are switched off for the device pass (the host pass
# does not know the feature and says so; that warning is harmless).
DEVICE = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src):
    out = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    path = os.path.join(CSRC, src)
    cmd = [HIPCC] + COMMON
    if src.endswith(".hip"):
        cmd += DEVICE
    else:
        cmd += ["-x", "c++"]
    cmd += ["-c", path, "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return out


def _build_marshal():
    # (to a new file, put in the old one's place: a process that has the old one loaded keeps it whole)
    out = MARSHAL + ".new"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-Wall", "-shared", "-I" + sysconfig.get_paths()["include"],
           os.path.join(CSRC, "marshal.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compiling marshal.cpp failed:\n" + r.stderr)
    if r.stderr.strip():
        sys.stderr.write(r.stderr)
    os.replace(out, MARSHAL)


def build(verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        marshal = ex.submit(_build_marshal)
        objs = list(ex.map(_compile, SOURCES))
        marshal.result()
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
