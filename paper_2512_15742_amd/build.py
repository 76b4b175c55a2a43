"""Builds libkan_mi355x.so (gfx950) in-tree with hipcc, and the extension module _kan_host.so (host
code of the binding's per-request calls) beside it with g++ against the installed torch.

    python -m paper_2512_15742_amd.build

Objects go to `_build/` at the repository root (not committed); the shared
library lands next to this file so that it travels with the source tree.
hipcc cross-compiles for gfx950 without a GPU being present.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libkan_mi355x.so")
HOST = os.path.join(HERE, "_kan_host.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed fp32 VALU forms are kept out of the generated code: some have given wrong results now and then
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]

# (source, object name, extra flags)
UNITS = [
    ("kan_api.hip", "kan_api.o", []),
    ("kan_misc.hip", "kan_misc.o", []),
    ("kan_mfma.hip", "kan_mfma.o", []),
    ("kan_mfma.hip", "kan_prep_rot.o", ["-DKAN_PREP_ROT=1"]),
    ("kan_stream.hip", "kan_stream.o", []),
    ("kan_wide.hip", "kan_wide.o", []),
    ("kan_wide.hip", "kan_wide_u32.o", ["-DKAN_WIDE_U32=1"]),
    ("kan_tail.hip", "kan_tail.o", []),
    ("kan_fused.hip", "kan_fused.o", []),
    ("kan_fused.hip", "kan_fused_chained.o", ["-DKAN_FUSED_CH=1"]),
    ("kan_fused_wave.hip", "kan_fused_wave.o", []),
    ("kan_fused_wave.hip", "kan_fused_wave_half.o", ["-DKAN_WAVE_HALF=1"]),
    ("kan_bucket.hip", "kan_bucket.o", []),
    ("kan_assign.hip", "kan_assign.o", []),
    ("kan_gather.hip", "kan_gather.o", []),
    ("kan_dense.hip", "kan_dense.o", []),
]


def _compile(unit, extra_flags):
    src, obj, flags = unit
    cmd = [HIPCC, *COMMON, *flags, *extra_flags, "-c", os.path.join(CSRC, src), "-o", os.path.join(BUILD, obj)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    return unit, r.returncode, r.stdout + r.stderr


def build(verbose: bool = True, extra_flags=(), jobs: int = 6) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        results = list(ex.map(lambda u: _compile(u, list(extra_flags)), UNITS))
    for unit, rc, out in results:
        noise = "unknown feature" in out or "not a recognized feature" in out
        if rc != 0 or (verbose and out.strip() and not noise):
            sys.stderr.write(f"[{unit[1]}] rc={rc}\n{out}\n")
        if rc != 0:
            raise RuntimeError(f"hipcc failed on {unit[0]} ({unit[1]})")
    objs = [os.path.join(BUILD, u[1]) for u in UNITS]
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    build_host()
    if verbose:
        print(f"built {LIB} and {HOST}")
    return LIB


def build_host() -> str:
    """The extension module: plain C++ against torch's headers and this library's C-ABI."""
    import sysconfig

    import torch
    t = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           "-isystem", os.path.join(t, "include"), "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "kan_host.cpp"), "-o", HOST, "-L" + os.path.join(t, "lib"), "-L" + HERE,
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on kan_host.cpp:\n" + r.stdout + r.stderr)
    return HOST


if __name__ == "__main__":
    build()
