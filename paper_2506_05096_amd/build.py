"""Builds libastraea.so (HIP, gfx950 only) next to this file."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
from pathlib import Path

PKG = Path(__file__).resolve().parent
ROOT = PKG.parent
CSRC = PKG / "csrc"
LIB = PKG / "libastraea.so"
OBJ = PKG / "_build"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # packed fp32 VALU forms are kept off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first 16 dwords of a kernel's arguments come in registers, set up with the wave, instead of by a load that it waits for: 0.2 - 0.3 us of a
    # launch; us a layer-step without / with: 2025 tokens at 30 % 49.8 / 48.4, 1055 x 211 x 16 32.5 / 30.0, block 1199 x 600 x 24 265.1 / 262.6
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-I", str(ROOT / "include"), "-I", str(CSRC),
]

# The attention's sweep: the time of a loop whose waves meet at a barrier every 200 instructions depends on where its branch targets lie in an
# instruction cache line.  All of them at the start of a line, same code otherwise, us: 35640 queries x 118800 keys x 24 heads 38440 ->
# 38278, 7020 x 17550 x 24 1175.4 -> 1173.3.
FILE_FLAGS = {"attn_bf16": ["-mllvm", "-align-all-nofallthru-blocks=6"]}


def sources():
    return sorted(CSRC.glob("*.hip"))


def _compile(src: Path) -> Path:
    obj = OBJ / (src.stem + ".o")
    subprocess.run([HIPCC, *FLAGS, *FILE_FLAGS.get(src.stem, []), "-c", str(src), "-o", str(obj)], check=True)
    return obj


def build(verbose: bool = True) -> Path:
    """Compile every .hip file and link the shared library.  Always rebuilds."""
    OBJ.mkdir(exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", str(LIB), *map(str, objs)], check=True)
    if verbose:
        print(f"built {LIB}")
    return LIB


def ensure_built() -> Path:
    """Build only when no library is present (tests, smoke and bench load what is there)."""
    if not LIB.exists():
        build()
    return LIB


if __name__ == "__main__":
    build()
