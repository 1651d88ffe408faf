"""Build the gfx950 shared library ``libmdeam.so`` in-tree with hipcc.

    python -m paper_1107_2619_amd.build

Every HIP source is compiled for gfx950 only, with packed FP32 instructions
disabled (``-packed-fp32-ops``): the mixed-precision path relies on plain
FP32 vector arithmetic.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmdeam.so")
SOURCES = ["kernels.hip", "kernels_global_f64.hip", "kernels_global_f64_multi.hip", "kernels_global_mixed.hip",
           "kernels_global_mixed_multi.hip", "kernels_build.hip", "kernels_brick.hip", "kernels_pairs.hip", "kernels_analysis.hip",
           "kernels_box.hip", "md_runtime.hip"]
ARCH = "gfx950"


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def flags() -> list[str]:
    return [
        f"--offload-arch={ARCH}",
        "-O3",
        "-std=c++17",
        "-fPIC",
        "-Wall",
        "-Wno-unused-function",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        f"-I{os.path.dirname(HERE)}",
    ]


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared library; return its path."""
    objs, procs = [], []
    for src in SOURCES:  # the translation units compile in parallel
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [hipcc(), *flags(), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd)))
        objs.append(obj)
    for cmd, proc in procs:
        if proc.wait() != 0:
            raise subprocess.CalledProcessError(proc.returncode, cmd)
    tmp = LIB + f".tmp{os.getpid()}"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
