"""Builds libwush.so (gfx950 only) in-tree with hipcc, and beside it libwush_probes.so, the
benchmark's measurement aids (MFMA-only and streaming kernels: not part of the layer path), and
_wush_call, the Python module of the per-step calls (where the running Python's headers are there).

Usage: python -m paper_2512_00956_amd.build
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libwush.so")
CALL_SRC = os.path.join(CSRC, "py_call.cpp")
# named for the Python it is built for: another one does not load it (and calls through ctypes)
CALL_LIB = os.path.join(HERE, "_wush_call" + sysconfig.get_config_var("EXT_SUFFIX"))
PROBES_SRC = os.path.join(HERE, "probes", "probes.hip")
PROBES_LIB = os.path.join(HERE, "libwush_probes.so")
SOURCES = ["wush_api.hip", "transform_quant.hip", "weight_prep.hip", "mxfp4_gemm.hip", "mxfp4_gemm_frag.hip", "mxfp4_gemm_canon.hip", "mxfp4_gemm_canon_stream.hip", "build_transforms.hip", "layer_decode.hip", "gptq_prep.hip", "nvfp4_quant.hip", "nvfp4_gemm.hip", "int4_quant.hip", "w4_gemm_skinny.hip"]

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed FP32 VALU ops stay disabled for every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc_path() -> str:
    p = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(p):
        raise RuntimeError("hipcc not found: the HIP library cannot be built")
    return p


def check_generated_code(hipcc: str, bdir: str) -> None:
    """What the kernels rely on in the generated code (build_checks.py) is verified on every build, with the flags of the build: the
    wait states behind matrix instructions in all of them, and what the MXFP4 GEMMs that issue their main-loop loads from inline asm need."""
    from .build_checks import check_gemm_canon_asm, check_gemm_frag_asm, check_lds_load_asm, check_mfma_result_waits
    more = {"mxfp4_gemm_frag.hip": (check_gemm_frag_asm, check_lds_load_asm),
            "mxfp4_gemm_canon.hip": (check_gemm_canon_asm, check_lds_load_asm)}
    procs = []
    for src in SOURCES:
        asm = os.path.join(bdir, src.replace(".hip", ".s"))
        cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-S", "--cuda-device-only", os.path.join(CSRC, src), "-o", asm]
        procs.append((src, asm, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    texts = {}
    for src, asm, p in procs:                       # all of them end before a check may raise
        out, _ = p.communicate()
        if p.returncode != 0:
            raise RuntimeError(f"hipcc -S failed on {src}:\n{out}")
        with open(asm) as f:
            texts[src] = f.read()
        os.remove(asm)
    for src, text in texts.items():
        for check in (check_mfma_result_waits, *more.get(src, ())):
            check(text)                             # raises InvariantError


def build_call_module() -> str | None:
    """The Python module of the per-step calls: host code only, finds libwush.so beside itself.  Needs the running Python's
    headers and g++; without them the binding makes the same calls through ctypes.  Returns its path, or None."""
    stale = os.path.join(HERE, "_wush_call.so")          # a module any Python would load
    if os.path.exists(stale):
        os.remove(stale)
    include, compiler = sysconfig.get_paths()["include"], shutil.which("g++")
    if compiler is None or not os.path.exists(os.path.join(include, "Python.h")):
        print("_wush_call is not built (no g++ or no Python.h): the per-step calls go through ctypes", file=sys.stderr)
        if os.path.exists(CALL_LIB):
            os.remove(CALL_LIB)                          # it belongs to an earlier libwush.so
        return None
    tmp = CALL_LIB + ".tmp"
    cmd = [compiler, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", include, "-I", os.path.join(ROOT, "include"),
           CALL_SRC, "-o", tmp, "-L", HERE, "-lwush", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on py_call.cpp:\n{r.stdout}")
    os.replace(tmp, CALL_LIB)
    return CALL_LIB


def build(verbose: bool = False) -> str:
    """Compile every kernel source and link libwush.so; returns its path."""
    hipcc = hipcc_path()
    objs = []
    procs = []
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(bdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    pobj = os.path.join(bdir, "probes.o")
    pcmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-c", PROBES_SRC, "-o", pobj]
    procs.append(("probes/probes.hip", subprocess.Popen(pcmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    check_generated_code(hipcc, bdir)
    for lib, lobjs in ((LIB, objs), (PROBES_LIB, [pobj])):
        tmp = lib + ".tmp"
        cmd = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", *lobjs, "-o", tmp]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{r.stdout}")
        os.replace(tmp, lib)
    build_call_module()
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
