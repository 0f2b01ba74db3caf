"""Compile the HIP sources into ``libsymph.so`` (gfx950 only), in-tree next to this file."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsymph.so")
# Python extension module: the attention call's marshalling (host code only).  The name says which interpreter it is for.
CALL_LIB = os.path.join(HERE, "_attn_call" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ("api.hip", "kv_migrate.hip", "prefill_attn.hip", "rows_attn.hip", "attn_static.hip", "kv_pool.cpp")  # the last one is host code only
# packed-fp32 instructions are switched off for every device compile
HIPCC_FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def build_attn_call() -> bool:
    """Compile the attention call's marshalling.  The binding does without it where the interpreter's headers or gcc are absent."""
    include = sysconfig.get_paths()["include"]
    for old in (CALL_LIB, os.path.join(HERE, "_attn_call.so")):  # (the second: a name that any interpreter would load)
        if os.path.exists(old):
            os.remove(old)
    if not os.path.exists(os.path.join(include, "Python.h")):
        print(f"[build] no Python.h in {include}: the attention call is marshalled in Python", file=sys.stderr)
        return False
    gcc = shutil.which("gcc")
    if gcc is None:
        print("[build] no gcc: the attention call is marshalled in Python", file=sys.stderr)
        return False
    tmp = CALL_LIB + f".tmp{os.getpid()}"
    subprocess.check_call([gcc, "-O2", "-std=c11", "-Wall", "-shared", "-fPIC", "-I", include, "-I",
                           os.path.join(ROOT, "include"), os.path.join(CSRC, "attn_call.c"), "-o", tmp])
    os.replace(tmp, CALL_LIB)
    return True


def build(verbose: bool = False) -> str:
    """Always recompiles; returns the path of the shared library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(build_dir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", os.path.join(CSRC, src),
               "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = False
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(ln for ln in out.splitlines() if "packed-fp32-ops" not in ln)
        if pr.returncode != 0:
            failed = True
            print(f"[build] {src} FAILED\n{out}", file=sys.stderr)
        elif out.strip() and verbose:
            print(out)
    if failed:
        raise RuntimeError("hipcc failed")
    build_attn_call()
    tmp = LIB + f".tmp{os.getpid()}"
    subprocess.check_call([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
