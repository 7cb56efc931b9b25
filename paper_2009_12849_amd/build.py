"""Build libmonc.so (HIP for gfx950) in-tree with hipcc.

    python -m paper_2009_12849_amd.build

Objects go to paper_2009_12849_amd/_build/, the library next to this file.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmonc.so")
SOURCES = ["kernels.hip", "tridiag.hip", "level.hip", "krylov.hip", "api.hip", "probe.hip", "launch_shape.cpp",
           "plan_math.cpp"]
# the FFT kernels' compile-time lengths, one object per group (kernels.h)
FFT_GROUPS = 8
# (source, object, extra flags)
UNITS = [("fft_inst.hip", f"fft_inst_{k}.o", [f"-DMONC_FFT_GROUP={k}"]) for k in range(FFT_GROUPS)] + [
    (s, os.path.splitext(s)[0] + ".o", []) for s in SOURCES]

# No packed FP32 instructions (v_pk_*_f32) in any HIP object.
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             # FP atomics as the hardware instructions (the library's atomics
             # only touch its callers' hipMalloc'd device buffers)
             "-munsafe-fp-atomics",
             "-Wno-unused-result"]


def hipcc() -> str:
    path = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(path):
        raise RuntimeError("hipcc not found")
    return path


def _compile(unit) -> str:
    src, obj, flags = unit
    obj = os.path.join(BUILD, obj)
    cmd = [hipcc()] + HIP_FLAGS + flags + ["-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".cpp"):
        cmd = [hipcc(), "-O3", "-std=c++17", "-fPIC", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile of {src} failed:\n{' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(len(UNITS), os.cpu_count() or 1)) as ex:
        objs = list(ex.map(_compile, UNITS))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
