"""Compile libdnslab.so for gfx950 with hipcc (in-tree, no JIT cache).

Every translation unit is compiled separately (in parallel) into
``_build/`` and linked into ``libdnslab.so`` next to this file.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdnslab.so")
SOURCES = ["api.hip", "stencil.hip", "fft.hip", "fft_split.hip", "fft_line.hip", "particles.hip", "postproc.hip"]
ARCH = "gfx950"

# Kernel instances of the FFT solves on register tiles, one object per real
# type, pass and range of the length tables: fft_split.h (23 x and 19 z
# lengths), fft_line.h (23 x lengths, 18 column lengths).
PARTS = [(src, f"{name}_{ax}{bits}_{h}", real, ax == "x", lo, hi)
         for src, name, axes in (("fft_split_part.hip", "split", (("x", (0, 8, 16, 23)), ("z", (0, 7, 13, 19)))),
                                 ("fft_line_part.hip", "line", (("x", (0, 12, 23)), ("c", (0, 10, 18)))))
         for bits, real in ((64, "double"), (32, "float"))
         for ax, cuts in axes
         for h, (lo, hi) in enumerate(zip(cuts, cuts[1:]))]

# Packed FP32 instructions are disabled for all device code.
HIPFLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function", "-Wno-unused-variable", "-Wno-unused-result",
            "-I", INCLUDE, "-I", CSRC]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    cc = hipcc()
    procs = []
    objs = []
    units = [(src, src.replace(".hip", ".o"), []) for src in SOURCES]
    units += [(src, fn + ".o",
               [f"-DDNSLAB_PART_FN={fn}", f"-DDNSLAB_PART_T={real}", f"-DDNSLAB_PART_X={int(x)}",
                f"-DDNSLAB_PART_LO={lo}", f"-DDNSLAB_PART_HI={hi}"]) for src, fn, real, x, lo, hi in PARTS]
    for src, o, defs in units:
        obj = os.path.join(BUILD, o)
        objs.append(obj)
        cmd = [cc, *HIPFLAGS, *defs, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    errors = []
    for src, p in procs:
        out, _ = p.communicate()
        text = out.decode(errors="replace")
        if p.returncode != 0:
            errors.append(f"--- {src} ---\n{text}")
        elif verbose and text.strip():
            print(text, flush=True)
    if errors:
        raise RuntimeError("hipcc failed:\n" + "\n".join(errors))
    tmp = LIB + ".tmp"
    cmd = [cc, "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", tmp]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout.decode(errors="replace"))
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
