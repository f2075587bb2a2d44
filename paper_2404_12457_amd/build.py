"""Build libragc.so (the C-ABI library) and libragc_calib.so (the benchmark's calibration
kernels) for gfx950 with hipcc, and the extension _calls (argument marshalling for Python), in-tree.

    python -m paper_2404_12457_amd.build

Cross-compiles without a GPU.  Objects go to csrc/_build/ (ignored), the library
to paper_2404_12457_amd/libragc.so.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libragc.so")
CALIB_LIB = os.path.join(HERE, "libragc_calib.so")
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))  # for this interpreter, host code only
SOURCES = ["ragc_api.cpp", "ragc_ctl.cpp", "kv_ops.hip", "attn_f32.hip", "attn_bf16.hip", "attn_bf16_rows.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
    # packed fp32 math is kept off on this target (see the build notes)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-inline-asm",
]


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(extra_flags=(), verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES + ["calib.hip"]))
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs[:-1]], check=True)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", CALIB_LIB, objs[-1]], check=True)
    headers = sysconfig.get_paths()["include"]
    if os.path.exists(os.path.join(headers, "Python.h")):
        subprocess.run(["hipcc", "-x", "c++", "-no-hip-rt", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", headers,
                        os.path.join(CSRC, "py_calls.cpp"), "-o", CALLS], check=True)
    else:
        sys.stderr.write(f"no Python.h in {headers}: {os.path.basename(CALLS)} is left out, calls go through ctypes\n")
    if verbose:
        print("built", LIB, "and", CALIB_LIB)
    return LIB


if __name__ == "__main__":
    build(sys.argv[1:], verbose=True)
