"""Build step of the HIP library: compiles ``csrc/`` into ``libnf.so`` (gfx950).

Run as ``python -m paper_2606_06720_amd.build_lib`` or through
``__graft_entry__.build()``.  It always recompiles.
"""

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libnf.so")

SOURCES = ["nf_loop_row64.hip", "nf_loop_row32.hip", "nf_loop_col64.hip", "nf_loop_col32.hip", "nf_team.hip",
           "nf_team64a.hip", "nf_team64b.hip", "nf_team32a.hip", "nf_team32b.hip", "nf_chip.hip", "nf_chip64a.hip",
           "nf_chip64b.hip", "nf_chip64c.hip", "nf_chip32a.hip", "nf_chip32b.hip", "nf_chip32c.hip", "nf_kernels.hip",
           "nf_kernels3d.hip", "nf_api.cpp", "nf_batch.cpp", "nf_noalloc.hip", "nf_tune.cpp"]

HIP_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # packed FP32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]


def hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose=False):
    objs = []
    cc = hipcc()
    tmp = LIB + ".tmp"
    procs = []
    # the translation units are independent: compile them concurrently
    for src in SOURCES:
        obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
        cmd = [cc, *HIP_FLAGS, "-I", INCLUDE, "-I", CSRC, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((subprocess.Popen(cmd), cmd))
        objs.append(obj)
    for pr, cmd in procs:
        if pr.wait() != 0:
            raise subprocess.CalledProcessError(pr.returncode, cmd)
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
