"""Builds the HIP library (libca_hip.so) in-tree with hipcc for gfx950.

    python -m paper_2403_19708_amd.build

hipcc cross-compiles without a GPU.  Packed-fp32 instruction selection is switched off for all
device code.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = ["ca_lib.hip", "ca_move.hip", "ca_attn_ref.hip", "ca_attn_dma.hip", "ca_attn_prerot.hip", "ca_attn_pp.hip", "ca_attn_decode.hip", "ca_attn_rows.hip",
           "ca_store.cpp"]   # the last one is host code only (placement manager)
LIB = os.path.join(HERE, "libca_hip.so")
BINDING_SRC = os.path.join(HERE, "csrc", "ca_binding.cpp")         # CPython module next to it, linked against it
BINDING = os.path.join(HERE, "_ca_native" + sysconfig.get_config_var("EXT_SUFFIX"))
PROBE_SRC = os.path.join(HERE, "csrc", "mfma_rate_probe.hip")   # stand-alone measurement aid the benchmark runs
PROBE = os.path.join(HERE, "mfma_rate_probe")

FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared", "-Wl,-soname,libca_hip.so",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-const-variable",
    # the LDS-direct loads set m0 in inline assembly and list it as clobbered; clang notes for every use that
    # m0 is a reserved register (the kernels use no other instruction that reads it)
    "-Wno-inline-asm",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def is_stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(BINDING):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(BINDING))
    deps = [os.path.join(HERE, "csrc", s) for s in SOURCES]
    deps += [BINDING_SRC, os.path.join(HERE, "csrc", "ca_internal.h"), os.path.join(HERE, "csrc", "ca_device.h"), os.path.join(ROOT, "include", "ca.h"),
             os.path.join(ROOT, "include", "ca_store.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def build(verbose: bool = True) -> str:
    """Compiles every HIP source into one shared library; always recompiles."""
    cmd = [hipcc()] + FLAGS + [os.path.join(HERE, "csrc", s) for s in SOURCES] + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"   # host pass does not know the GPU feature
    for line in (proc.stdout + proc.stderr).splitlines():
        if noise not in line and verbose:
            print(line)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed")
    cmd = [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I" + sysconfig.get_paths()["include"], BINDING_SRC,
           LIB, "-Wl,-rpath,$ORIGIN", "-o", BINDING]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        print(proc.stderr)
        raise RuntimeError("g++ failed (ca_binding)")
    cmd = [hipcc(), "-O3", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           PROBE_SRC, "-o", PROBE]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        print(proc.stderr)
        raise RuntimeError("hipcc failed (mfma_rate_probe)")
    return LIB


if __name__ == "__main__":
    build()
    print("built", LIB)
    sys.exit(0)
