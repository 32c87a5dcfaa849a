"""Builds libparse.so (the C-ABI library) from the HIP sources with hipcc for gfx950, and the module _calls (its calls for Python) with g++."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libparse.so")
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))      # CPython module of the step's calls; another Python does not take it
SOURCES = ["api.hip", "route.hip", "cache.hip", "pack.hip", "bucket.hip", "forward_f32.hip",
           "prefill_bf16.hip", "prefill_split_bf16.hip", "prefill_lds_bf16.hip", "plan.hip", "decode_bf16.hip", "decode_wide_bf16.hip", "decode_static.hip", "forward.hip", "ranks.hip", "train.hip", "peaks.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-I" + INCLUDE, "-I" + CSRC,
         # packed-fp32 instruction selection is switched off for all device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = True, jobs: int = 8) -> str:
    """Compiles every source (always, also when a library is already there) and links libparse.so."""
    cc = hipcc()
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        extra = os.environ.get("PARSE_HIPCC_FLAGS", "").split()   # e.g. diagnostics switches while tuning
        cmd = [cc, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if len(procs) >= jobs:
            _drain(procs, verbose)
    _drain(procs, verbose)
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    out = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if out.returncode != 0:
        raise RuntimeError("link failed:\n" + out.stdout)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-I" + INCLUDE,
           "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "calls.cpp"), "-o", CALLS, "-L" + HERE, "-l:libparse.so",
           "-Wl,-rpath,$ORIGIN"]
    out = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if out.returncode != 0:
        raise RuntimeError("g++ failed on calls.cpp:\n" + out.stdout)
    if verbose:
        if out.stdout.strip():
            print(out.stdout)
        print("built", LIB, CALLS)
    return LIB


def _drain(procs, verbose):
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        text = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{text}")
        if verbose and text.strip():
            print(text)


if __name__ == "__main__":
    build()
    sys.exit(0)
