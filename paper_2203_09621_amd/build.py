"""Build libdmpt.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2203_09621_amd.build

Every call recompiles.  The shared library lands next to this file.
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
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libdmpt.so")
SOURCES = ["kernels_gemm.hip", "kernels_layer.hip", "kernels_adjoint.hip", "dmpt_api.hip",
           "dmpt_batch.hip", "dmpt_ortho.hip", "kernels_tiny.hip"]
ARCH = "gfx950"


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; the HIP library cannot be built")
    return exe


def _flags():
    return ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-I", INCLUDE, "-I", CSRC,
            # packed FP32 VALU forms stay disabled (hipcc flag for the device pass)
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            # Loops start on an instruction cache line.  The product kernels run one or
            # two waves per SIMD, so nothing hides a fetch: a main loop whose first four
            # bytes were the last of a line cost 4% (26.9 against 25.9 ms per launch of
            # the 256-row kernel at N = 16384), and where a loop lands would otherwise
            # change with any edit of the file.
            "-falign-loops=64",
            "-Wno-unused-command-line-argument"]


def build(verbose: bool = False) -> str:
    obj_dir = os.path.join(HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    cc = hipcc()

    def compile_one(src):
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        cmd = [cc, *_flags(), "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
        if verbose:
            sys.stderr.write(r.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [cc, "--offload-arch=" + ARCH, "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
