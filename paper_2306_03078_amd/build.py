"""Builds libspqr.so (HIP, gfx950) in-tree with hipcc: one object per source, compiled side by side, then linked; and the
extension module through which Python calls it (host code only)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libspqr.so")
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["spqr_pack.cpp", "spqr_api.hip", "spqr_dispatch.hip", "spqr_gemv.hip", "spqr_gemv_l1.hip", "spqr_gemv_l1w.hip", "spqr_gemv_l2.hip", "spqr_gemv_l3.hip", "spqr_mfma.hip", "spqr_prompt.hip", "spqr_prefill.hip", "spqr_misc.hip", "spqr_encode.hip", "spqr_factor.hip", "spqr_order.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # packed-FP32 VALU forms are kept out of the generated code on purpose
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _run(cmd, verbose):
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(" ".join(cmd))
        print(res.stdout)
        print("\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l))
    if res.returncode != 0:
        raise RuntimeError("the compiler failed: " + " ".join(cmd[-3:]))


def build_library(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    objs = [os.path.join(OBJ, os.path.splitext(s)[0] + ".o") for s in SOURCES]
    jobs = [[hipcc, *FLAGS, "-c", "-o", o, os.path.join(CSRC, s)] for s, o in zip(SOURCES, objs)]
    with ThreadPoolExecutor(max_workers=min(len(jobs), os.cpu_count() or 1, 8)) as pool:
        list(pool.map(lambda c: _run(c, verbose), jobs))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], verbose)
    calls = calls_command()
    if calls is not None:
        _run(calls, verbose)
    else:                        # nor one of an earlier build
        if os.path.exists(CALLS):
            os.remove(CALLS)
        print("no C compiler or no Python.h: Python calls the library through ctypes", file=sys.stderr)
    return LIB


def calls_command():
    """The command that builds the extension module, None where there is no C compiler or no Python.h: the binding does without."""
    include = sysconfig.get_paths()["include"]
    cc = next(filter(None, map(shutil.which, ["gcc", "cc", "clang"])), None)
    if cc is None or not os.path.exists(os.path.join(include, "Python.h")):
        return None
    return [cc, "-O2", "-Wall", "-shared", "-fPIC", "-I" + include, "-o", CALLS, os.path.join(CSRC, "spqr_calls.c")]


if __name__ == "__main__":
    print(build_library(verbose=True))
