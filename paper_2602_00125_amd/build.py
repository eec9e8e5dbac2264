"""Build libminitensor_hip.so (in-tree, gfx950 only) with hipcc.

Every HIP source is compiled for gfx950 with packed-fp32 instruction
selection disabled; the host sources go through the same driver. The result
sits next to this file, where ``binding`` loads it, with the binding's own
native module beside it.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libminitensor_hip.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

SOURCES = ["gemm_f32.hip", "gemm_bf16.hip", "reduce.hip", "elementwise.hip", "conv.hip", "noalloc.hip",
           "shape.cpp", "capi.cpp", "conv_host.cpp"]
# what is compiled: (source, extra flags); the fp32 products take most of the
# time and compile in parts, side by side
UNITS = ([("gemm_f32.hip", [f"-DMT_F32_PART={n}"]) for n in (3, 4, 1, 2, 6, 5)] +
         [(s, []) for s in SOURCES if s != "gemm_f32.hip"])
COMMON = ["-std=c++17", "-O3", "-fPIC", "-Wall", "-Wno-unused-result",
          f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-I", os.path.join(HERE, "..", "include")]


def _compile(src: str, objdir: str, extra: list[str], tag: str = "") -> str:
    obj = os.path.join(objdir, os.path.basename(src) + tag + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    cmd = [HIPCC, *COMMON, *extra, *lang, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def _build_marshal() -> None:
    """The native half of binding.py: a CPython module, host code only."""
    out = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
    tmp = out + ".tmp"
    cmd = [os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-fPIC", "-shared", "-Wall",
           "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "pymarshal.cpp"), "-o", tmp, "-ldl"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, out)


def build(extra: list[str] | None = None, verbose: bool = False) -> str:
    extra = list(extra or [])
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(UNITS))) as ex:
        objs = list(ex.map(lambda u: _compile(u[1][0], objdir, extra + u[1][1], f".{u[0]}"), enumerate(UNITS)))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, OUT)
    _build_marshal()
    if verbose:
        print(f"built {OUT}")
    return OUT


if __name__ == "__main__":
    build(sys.argv[1:], verbose=True)
