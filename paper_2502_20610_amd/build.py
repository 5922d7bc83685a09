"""Build libfdtd.so (hand-written HIP for gfx950) in-tree.

hipcc flags:
  --offload-arch=gfx950        MI355X only
  -O3 -ffp-contract=off        no fused multiply-add: every operation of the
                               update rounds separately, as the update
                               equations are written
  -target-feature -packed-fp32-ops
                               no packed FP32 instructions
Denormals stay IEEE (no -ffast-math, no flush-to-zero).
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfdtd.so")
SOURCES = ["systolic.hip", "sweep.hip", "sweep_batch.hip", "sweep_adjoint.hip", "fdtd_api.hip", "plain.hip",
           "adjoint.hip", "invariants.hip", "materials.hip", "autotune.hip", "plan.cpp", "sweep_plan.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-Wall", "-Wno-unused-function"]


def build(verbose: bool = False) -> str:
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = [os.path.join(objdir, os.path.splitext(src)[0] + ".o") for src in SOURCES]

    def compile_one(src, obj):
        cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            sys.stderr.write(err + "\n")
            raise RuntimeError("hipcc failed on %s" % src)
        if verbose and err.strip():
            sys.stderr.write(err + "\n")

    with ThreadPoolExecutor(4) as pool:
        list(pool.map(compile_one, SOURCES, objs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", tmp]
    subprocess.run(cmd, check=True, capture_output=not verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
