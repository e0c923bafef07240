"""Build libgeonav.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libgeonav.so")
SOURCES = ["geonav_kernels.hip", "geonav_abi.cpp"]
PARTS = {"geonav_kernels.hip": 5}  # objects a source is compiled to, by its sections (GEONAV_PART)
HEADERS = ["geonav_device.hpp", "geonav_internal.hpp"]

ARCH = os.environ.get("GEONAV_ARCH", "gfx950")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # contract a*b+c only within one source expression: results do not depend
    # on how the surrounding code is inlined or scheduled
    "-ffp-contract=on",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    f"-I{INCLUDE}", f"-I{CSRC}",
]


def build(verbose: bool = False) -> str:
    """Compile every source, the objects side by side, and link libgeonav.so
    (always rebuilds)."""
    objs, cmds = [], []
    bdir = os.path.join(PKG, "_build")
    os.makedirs(bdir, exist_ok=True)
    for src in SOURCES:
        parts = PARTS.get(src, 0)
        for part in range(1, parts + 1) if parts else [0]:
            obj = os.path.join(bdir, os.path.splitext(src)[0] + (str(part) if part else "") + ".o")
            cmd = ["hipcc", "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj] + FLAGS
            cmds.append(cmd + ([f"-DGEONAV_PART={part}"] if part else []))
            objs.append(obj)
            if verbose:
                print(" ".join(cmds[-1]), flush=True)
    procs = [subprocess.Popen(cmd) for cmd in cmds]
    codes = [p.wait() for p in procs]  # (all of them, so that none outlives a failure)
    for cmd, code in zip(cmds, codes):
        if code:
            raise subprocess.CalledProcessError(code, cmd)
    tmp = LIB + ".tmp"
    cmd = ["hipcc", "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, f) for f in SOURCES + HEADERS] + [os.path.join(INCLUDE, "geonav.h")]
    return any(os.path.getmtime(d) > t for d in deps)


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
