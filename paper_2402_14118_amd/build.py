"""Builds the HIP library in-tree (gfx950 only).  Cross-compiles without a GPU."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libmmm_hip.so")
NATIVE = os.path.join(PKG, "_mmm_native.so")       # CPython entry points, linked against the library
NATIVE_SOURCE = os.path.join(CSRC, "mmm_python.cpp")
SOURCES = ["mmm_api.hip", "mmm_build.hip", "mmm_matmul.hip", "mmm_pairs.hip"]
HEADERS = [os.path.join(CSRC, "mmm_internal.h"), os.path.join(ROOT, "include", "mmm.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed fp32 VALU forms are kept off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(NATIVE):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(NATIVE))
    deps = [os.path.join(CSRC, s) for s in SOURCES] + HEADERS + [NATIVE_SOURCE]
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every source and link libmmm_hip.so and the CPython entry points next to this file."""
    if not force and not stale():
        return LIB
    objs = []
    procs = []
    for s in SOURCES:
        obj = os.path.join(CSRC, s.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c",
               os.path.join(CSRC, s), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((s, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = False
    for s, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode != 0:
            failed = True
            sys.stderr.write(f"--- {s} failed ---\n{out}\n")
        elif verbose and out:
            print(out)
    if failed:
        raise RuntimeError("hipcc failed")
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-Wl,-soname,libmmm_hip.so", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    cmd = [CXX, "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I", os.path.join(ROOT, "include"),
           "-I", sysconfig.get_paths()["include"], NATIVE_SOURCE, "-o", NATIVE, "-L", PKG, "-l:libmmm_hip.so", "-Wl,-rpath,$ORIGIN"]
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
