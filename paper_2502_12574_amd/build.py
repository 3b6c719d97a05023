"""Compile the HIP sources into paper_2502_12574_amd/libheadinfer.so (gfx950 only), and the native call marshalling for Python."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libheadinfer.so")
PYCALL = os.path.join(HERE, "_pycall" + sysconfig.get_config_var("EXT_SUFFIX"))     # native marshalling for binding.py (host code)
SOURCES = ["hi_plan.cpp", "hi_ctx.hip", "hi_decode.hip", "hi_prefill.hip", "hi_proj.hip", "hi_kvq.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 vector ops are switched off for every device translation unit
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def build(verbose: bool = False) -> str:
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc(), *HIPCC_FLAGS, "-x", "hip", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
               "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    os.replace(tmp, LIB)
    build_pycall()
    return LIB


def build_pycall() -> str | None:
    """The native marshalling for this interpreter, where a host compiler and Python's headers are there (binding.py does without)."""
    if os.path.exists(PYCALL):
        os.remove(PYCALL)
    gxx, headers = shutil.which("g++") or shutil.which("c++"), sysconfig.get_paths()["include"]
    if gxx is None or not os.path.exists(os.path.join(headers, "Python.h")):
        print("no host compiler or no Python.h: every call from Python will go through ctypes (2 us more for each call of a token)")
        return None
    tmp = PYCALL + ".tmp"
    cmd = [gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-I", headers, "-I", os.path.join(ROOT, "include"),
           os.path.join(CSRC, "hi_pycall.cpp"), "-o", tmp]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("the host compiler failed on hi_pycall.cpp:\n" + r.stdout)
    os.replace(tmp, PYCALL)
    return PYCALL


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
