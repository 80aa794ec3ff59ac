"""Builds libentmax_attn.so (the HIP kernels plus the C ABI) for gfx950.

    python paper_2502_12082_amd/build.py        # from the repository root

Every .hip file under csrc/ is compiled with hipcc into _build/, in parallel
(the solver in parts), and linked into paper_2502_12082_amd/libentmax_attn.so next to this file.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build", "entmax_attn")
LIB = os.path.join(HERE, "libentmax_attn.so")
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    "--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall",
    # fp32 d=128 variants cannot reach the two-waves-per-SIMD target the bf16
    # ones are built for; the compiler reports that per instantiation
    "-Wno-pass-failed",
    # no packed fp32 VALU instructions in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]
# Files compiled in several parts, in parallel: (macro, number of parts).
PARTS = {"ea_tau.hip": ("EA_TAU_PART", 5)}


def _units():
    """(source, object, extra flags) of every translation unit, the files with
    several parts (the longest to compile) first."""
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")),
                  key=lambda s: (os.path.basename(s) not in PARTS, s))
    for src in srcs:
        name = os.path.basename(src)
        macro, parts = PARTS.get(name, (None, 1))
        for i in range(parts):
            if macro:
                yield src, os.path.join(BUILD, "%s.%d.o" % (name, i)), ["-D%s=%d" % (macro, i)]
            else:
                yield src, os.path.join(BUILD, name + ".o"), []


def _compile(unit) -> str:
    src, obj, flags = unit
    cmd = [HIPCC] + CFLAGS + flags + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj


def build(jobs: int | None = None) -> str:
    os.makedirs(BUILD, exist_ok=True)
    units = list(_units())
    jobs = jobs or min(len(units), max(1, (os.cpu_count() or 2)))
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, units))
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
