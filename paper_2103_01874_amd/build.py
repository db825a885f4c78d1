"""Build libppe.so (HIP, gfx950) in-tree with hipcc.

Usage: python -m paper_2103_01874_amd.build   (or call build()).
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libppe.so")
OBJ = os.path.join(HERE, "_build")
HOSTCHECK = os.path.join(HERE, "libppe_hostcheck.so")

HIP_FLAGS = [
    "-O3",
    "-std=c++17",
    "--offload-arch=gfx950",
    "-fPIC",
    # no packed-FP32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libppe.so)")


def _run(cmd, what, verbose=False):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed building {what}")


def _compile(src: str, out: str, extra=(), verbose=False):
    tmp = out + ".tmp"
    _run([hipcc(), *HIP_FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC, src, "-o", tmp],
         os.path.basename(out), verbose)
    os.replace(tmp, out)
    return out


def build(verbose: bool = False) -> str:
    """Compile libppe.so (the library) and libppe_hostcheck.so (CPU test support).

    The library's translation units -- ppe_lib.hip and, per spectrum precision
    and group of transform lengths, ppe_fft.hip -- compile side by side."""
    os.makedirs(OBJ, exist_ok=True)
    units = [("ppe_lib.hip", "ppe_lib.o", ())]
    units += [("ppe_fft.hip", f"ppe_fft_{ts}{grp}.o", (f"-DPPE_FFT_GROUP={grp}", f"-DPPE_FFT_TS={ts}"))
              for grp in range(5) for ts in ("double", "float")]
    with ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as ex:
        objs = [ex.submit(_compile, os.path.join(CSRC, src), os.path.join(OBJ, out), ("-c", *defs), verbose)
                for src, out, defs in units]
        host = ex.submit(_compile, os.path.join(CSRC, "hostcheck.cpp"), HOSTCHECK, ("-shared", "-x", "hip"), verbose)
        objs = [o.result() for o in objs]
        host.result()
    tmp = LIB + ".tmp"
    _run([hipcc(), *HIP_FLAGS, "-shared", *objs, "-o", tmp], os.path.basename(LIB), verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
