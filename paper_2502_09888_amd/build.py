"""Build libclimber.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2502_09888_amd.build

Each .hip file is compiled to an object next to it and the objects are linked into
``paper_2502_09888_amd/libclimber.so``; csrc/binding.c becomes the extension module ``_native`` beside it, named for the
interpreter that builds it.  Packed-FP32 instruction selection is switched off for all device code.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from importlib.machinery import EXTENSION_SUFFIXES

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libclimber.so")
NATIVE = os.path.join(HERE, "_native" + EXTENSION_SUFFIXES[0])
SOURCES = ["climber_api.hip", "attn_bf16.hip", "attn_wave_bf16.hip", "attn_split_bf16.hip", "attn_bias_bf16.hip", "attn_f32.hip", "attn_tile_f32.hip", "kv_cache.hip", "stack.hip",
           "gemm_bf16.hip", "gemm_small_bf16.hip", "gemm_resident_bf16.hip", "layer_tail_bf16.hip", "layer_head_bf16.hip", "rowwise.hip", "hist_fused_bf16.hip", "check.hip", "bgf.hip", "bgf_front_bf16.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def _stale(obj: str, src: str) -> bool:
    if not os.path.exists(obj):
        return True
    t = os.path.getmtime(obj)
    deps = [src] + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    deps.append(os.path.join(HERE, "..", "include", "climber.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = False, verbose: bool = False) -> str:
    hipcc = _hipcc()

    def compile_one(name):
        src = os.path.join(CSRC, name)
        obj = os.path.join(CSRC, name.replace(".hip", ".o"))
        if force or _stale(obj, src):
            cmd = [hipcc, *FLAGS, "-c", src, "-o", obj]
            r = subprocess.run(cmd, capture_output=True, text=True)
            err = "\n".join(l for l in r.stderr.splitlines()
                            if "packed-fp32-ops" not in l)
            if r.returncode != 0:
                raise RuntimeError(f"hipcc failed on {name}:\n{err}")
            if verbose and err.strip():
                print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    binding = os.path.join(CSRC, "binding.c")
    if force or _stale(NATIVE, binding):
        subprocess.check_call([os.environ.get("CC", "gcc"), "-O2", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"],
                               binding, "-o", NATIVE])
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
