"""Compile libflatquant.so (gfx950) and the extension module _fqcall in-tree with hipcc.  `python -m paper_2410_09426_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libflatquant.so")
# CPython calls of the library's entry points: host code that links nothing, for the interpreter that builds it (its name says which)
CALLS = os.path.join(PKG, "_fqcall" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["fq_api.hip", "fq_transform_quant.hip", "fq_tq_fast.hip", "fq_tq_wave.hip", "fq_tq_rows.hip", "fq_kv.hip", "fq_dequant.hip", "fq_probe.hip", "fq_gemm.hip", "fq_gemm_mx.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function",
         # keep hipcc from forming packed-fp32 VALU ops from scalar float code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


# Per-file additions.  The KV kernel's min/max chains run on MFMA results: without the promise that they are not NaN
# the compiler quiets every operand first (one extra instruction per element).  Inputs are finite by contract.
# The wave-per-token kernel takes plain arguments in the order it needs them; the first 14 dwords are delivered in
# registers at wave start (kernel-argument preloading), which takes a scalar-memory round trip off the front of every wave.
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]
FILE_FLAGS = {"fq_kv.hip": ["-fno-honor-nans"], "fq_tq_wave.hip": PRELOAD, "fq_gemm.hip": PRELOAD, "fq_gemm_mx.hip": PRELOAD}


def link(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    if verbose and r.stdout.strip():
        print(r.stdout.strip())


def build(verbose: bool = True, extra_flags=()) -> str:
    objs = []
    procs = []
    for s in SOURCES:
        o = os.path.join(CSRC, s.replace(".hip", ".o"))
        objs.append(o)
        cmd = [hipcc(), *FLAGS, *FILE_FLAGS.get(s, []), *extra_flags, "-c", os.path.join(CSRC, s), "-o", o]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((s, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for s, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {s}:\n{out}")
        if verbose and out.strip():
            print(out)
    link([hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB], verbose)
    untagged = os.path.join(PKG, "_fqcall.so")   # of an earlier build: any interpreter would take it
    if os.path.exists(untagged):
        os.remove(untagged)
    link([hipcc(), "-x", "c++", "-O2", "-std=c++17", "-Wall", "-fPIC", "-shared", "-no-hip-rt", "-I" + sysconfig.get_paths()["include"],
          os.path.join(CSRC, "fq_python.cpp"), "-o", CALLS], verbose)
    return LIB


if __name__ == "__main__":
    print(build(extra_flags=sys.argv[1:]))
