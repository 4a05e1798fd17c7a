"""Build libkia.so (gfx950) from csrc/ with hipcc, in-tree.

Every HIP source is compiled for gfx950 only, with packed-fp32 instruction
selection disabled and hardware float atomics enabled (device buffers are
ordinary coarse-grained allocations). Usage: ``python -m
paper_2609_33591_amd.build`` or ``build()`` from Python.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libkia.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
HEADS = (16, 32, 64, 128)
# object -> its compilations (source, extra flags): the kernels that are
# instantiated for every operator are compiled once per head dimension, in
# parallel, and joined into one relocatable object
OBJECTS = {
    "kia_abi.o": [("kia_abi.hip", [])],
    "kia_fwd.o": [("kia_fwd.hip", [f"-DKIA_HEAD={d}"]) for d in HEADS] + [("kia_debug.hip", [])],
    "kia_bwd.o": [("kia_bwd.hip", [f"-DKIA_HEAD={d}"]) for d in HEADS],
    "kia_bf16.o": [("kia_bf16.hip", [])],
}
# (source, flags, object file) of every compilation
UNITS = [(src, flags, obj if len(parts) == 1 else f"{obj[:-2]}_{i}.o")
         for obj, parts in OBJECTS.items() for i, (src, flags) in enumerate(parts)]
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
         "-munsafe-fp-atomics",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _run(cmd, what) -> None:
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{res.stderr}")


def _compile(unit) -> None:
    src, flags, obj = unit
    _run([HIPCC, *FLAGS, *flags, "-c", os.path.join(CSRC, src), "-o", os.path.join(BUILD, obj)],
         f"hipcc {src} {flags}")


def link() -> None:
    for obj, parts in OBJECTS.items():
        if len(parts) > 1:
            units = [os.path.join(BUILD, f"{obj[:-2]}_{i}.o") for i in range(len(parts))]
            _run(["ld", "-r", *units, "-o", os.path.join(BUILD, obj)], "ld -r")
    tmp = LIB + ".tmp"
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC",
          *(os.path.join(BUILD, o) for o in OBJECTS), "-o", tmp], "link")
    os.replace(tmp, LIB)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(len(UNITS), os.cpu_count() or 1)) as ex:
        list(ex.map(_compile, UNITS))
    link()
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
