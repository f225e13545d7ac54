"""Builds libmlkv.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
KERNELS = os.path.join(CSRC, "mlkv_kernels.hip")
# the row maps of mlkv_kernels.h (MLKV_MAPS), one compilation of mlkv_kernels.hip each, the slowest first
MAPS = ("MapD1024", "MapD512", "MapD256", "MapD128", "MapD64", "MapD32", "MapD16", "MapD3")
UNITS = [(KERNELS, m) for m in MAPS] + [(os.path.join(CSRC, f), None)
                                       for f in ("mlkv_kernels.hip", "mlkv_api.hip", "mlkv_tier.hip")]
LIB = os.path.join(HERE, "libmlkv.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # IEEE fp32: no contraction into fused multiply-adds, correctly rounded
    # division and square root
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    # no packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-const-variable",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _run(cmd: list[str]) -> str:
    """Runs a compiler command; returns what it printed, raises if it failed."""
    r = subprocess.run(cmd, capture_output=True, text=True)
    said = "\n".join(ln for ln in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in ln and ln.strip())
    if r.returncode != 0:
        sys.stderr.write(said + "\n")
        raise RuntimeError(f"hipcc failed with code {r.returncode}")
    return said


def build(verbose: bool = False) -> str:
    if verbose:
        print(" ".join([HIPCC, *FLAGS, "-c", "[-DMLKV_MAP=<map>]", CSRC + "/*.hip"]), flush=True)
    with tempfile.TemporaryDirectory() as tmp:
        def unit(i: int) -> str:
            src, row_map = UNITS[i]
            return _run([HIPCC, *FLAGS, *([f"-DMLKV_MAP={row_map}"] if row_map else []), "-c", src, "-o",
                         os.path.join(tmp, f"{i}.o")])

        with ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            said = list(pool.map(unit, range(len(UNITS))))
        said.append(_run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB + ".tmp",
                          *(os.path.join(tmp, f"{i}.o") for i in range(len(UNITS)))]))
    if verbose and any(said):
        print("\n".join(x for x in said if x))
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
