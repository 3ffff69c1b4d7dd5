"""Builds libgbmuf.so (gfx950) in-tree with hipcc.  Run as ``python -m paper_1909_09010_amd.build``."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libgbmuf.so")
# (source, defines): the fused kernel's shapes are compiled in five parts, each with plain and streamed accesses and for tiles in stretches
UNITS = [("gbmuf_sync.hip", [f"-DGBMUF_PART={i}", f"-DGBMUF_POLICY={j}"]) for i in (4, 3, 2, 0, 1) for j in (0, 1, 2)] + [
    ("gbmuf_plan.hip", []), ("gbmuf_kernels.hip", [])]

# -ffp-contract=off: the method's fp32 arithmetic rounds every multiply and add separately.
# The packed-fp32 feature is switched off on purpose (scalar fp32 VALU ops only).
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def build_library(verbose: bool = True, extra_flags=()) -> str:
    """Compiles every HIP source into paper_1909_09010_amd/libgbmuf.so (always recompiles), the
    objects side by side."""
    flags = [f for f in HIPCC_FLAGS if f != "-shared"] + list(extra_flags)
    with tempfile.TemporaryDirectory(prefix="gbmuf_build_") as tmp:
        objects, commands = [], []
        for src, define in UNITS:
            obj = os.path.join(tmp, f"{len(objects)}.o")
            objects.append(obj)
            commands.append([hipcc(), *flags, *define, "-c", "-o", obj, os.path.join(CSRC, src)])
        if verbose:
            for cmd in commands:
                print(" ".join(cmd), flush=True)
        running = [subprocess.Popen(cmd, cwd=CSRC) for cmd in commands]
        for cmd, status in [(cmd, p.wait()) for cmd, p in zip(commands, running)]:
            if status != 0:
                raise subprocess.CalledProcessError(status, cmd)
        subprocess.run([hipcc(), "--offload-arch=gfx950", "-fPIC", "-shared", "-o", LIB_PATH, *objects], check=True, cwd=CSRC)
    return LIB_PATH


if __name__ == "__main__":
    build_library(extra_flags=sys.argv[1:])
