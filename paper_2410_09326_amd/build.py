"""Builds libqops.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
OUT = os.path.join(HERE, "libqops.so")
OBJ = os.path.join(HERE, "_build")

SOURCES = ["kernels.hip", "regtile.hip", "mlp.hip", "planner.cpp", "runtime.cpp", "costmodel.cpp", "profile.cpp", "batch.cpp", "readout.hip", "fold.cpp",
           "noalloc.hip", "tier.cpp"]
# register tile variants (precision, register bits, wave bits): one object
# each, as in QOPS_TILE_VARIANTS of regtile.hpp
# The operation loop branches on wave-uniform values only; structurizing those
# branches would pass the whole tile through merge blocks that copy it.
REG_TILE_FLAGS = ["-mllvm", "-structurizecfg-skip-uniform-regions=true"]
REG_TILES = [(t, r, w) for r, ws in ((4, (3, 2, 0)), (3, (3, 2))) for t in ("double", "float") for w in ws]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no packed FP32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # keep register arrays in VGPRs (common-code sinking across switch cases
    # turns constant register indices into dynamic ones)
    "-mllvm", "-simplifycfg-sink-common=false",
    "-I", os.path.join(ROOT, "include"),
    "-Wno-unused-command-line-argument",
]


def _compile(unit) -> str:
    src, defines, name = unit
    obj = os.path.join(OBJ, name + ".o")
    path = os.path.join(CSRC, src)
    cmd = [HIPCC] + FLAGS + defines + ["-c", path, "-o", obj]
    if src.endswith(".cpp"):
        cmd = [HIPCC] + [f for f in FLAGS if f != "--offload-arch=gfx950"] + ["-x", "hip", "--offload-arch=gfx950", "-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    return obj


def units():
    """(source, defines, object name) of every object, the slowest first."""
    u = [("regtile.hip", REG_TILE_FLAGS + [f"-DQOPS_RT_T={t}", f"-DQOPS_RT_R={r}", f"-DQOPS_RT_W={w}"],
          f"regtile_{t}_{r}_{w}.hip") for t, r, w in REG_TILES]
    return [(SOURCES[0], [], SOURCES[0])] + u + [(s, [], s) for s in SOURCES[1:]]


def build(jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, units()))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link failed")
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build())
