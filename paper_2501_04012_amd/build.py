"""Builds libflexdenoise.so for gfx950 with hipcc, and the CPython side of the binding, in-tree.

    python -m paper_2501_04012_amd.build [--force]
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libflexdenoise.so")
SOURCES = ["flexdenoise.hip", "elementwise.hip", "gemm.hip", "attention.hip", "chain.hip", "cache.hip", "microbench.hip"]
# the cache calls as CPython functions (host only), for the interpreter that builds them
PYCALL_PATH = os.path.join(HERE, "_pycall" + sysconfig.get_config_var("EXT_SUFFIX"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the packed-fp32 feature and says so; that line is noise
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("command failed: " + " ".join(cmd) + "\n" + out)
    return out


def build(force: bool = True, verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    headers = [os.path.join(CSRC, "common.h"), os.path.join(HERE, "..", "include", "flexdenoise.h")]
    newest_hdr = max(os.path.getmtime(h) for h in headers)

    def compile_one(src):
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
        if not force and os.path.exists(o) and os.path.getmtime(o) > max(os.path.getmtime(s), newest_hdr):
            return o, ""
        return o, _run([HIPCC, *FLAGS, "-c", s, "-o", o])

    with ThreadPoolExecutor(max_workers=6) as ex:
        results = list(ex.map(compile_one, SOURCES))
    for _, log in results:
        if verbose and log.strip():
            print(log)
    objs = [o for o, _ in results]
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs])
    src = os.path.join(CSRC, "pycall.cpp")
    if force or not os.path.exists(PYCALL_PATH) or os.path.getmtime(PYCALL_PATH) < max(os.path.getmtime(src), newest_hdr):
        for old in (PYCALL_PATH, os.path.join(os.path.dirname(PYCALL_PATH), "_pycall.so")):      # (any interpreter would load the second)
            if os.path.exists(old):
                os.remove(old)
        try:
            _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                  "-I" + sysconfig.get_paths()["include"], src, "-o", PYCALL_PATH])
        except (OSError, RuntimeError) as e:             # no host compiler, or no headers of this interpreter
            print(f"{os.path.basename(PYCALL_PATH)} not built, the cache calls go through ctypes: {e}", file=sys.stderr)
    return LIB_PATH


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
