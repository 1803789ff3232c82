"""Builds libmclya.so, the HIP library for gfx950 (MI355X).

Every source under csrc/ is compiled by hipcc for gfx950 only, in parallel,
then linked into a shared library next to this file. Packed FP32 instructions
are disabled and floating-point contraction is limited to single expressions,
so every packet's arithmetic is the same whichever kernel runs it.
"""
import concurrent.futures as cf
import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmclya.so")
LIB_ENDS = os.path.join(HERE, "libmclya_ends.so")   # --count-ends
OBJ = os.path.join(ROOT, "_build", "mclya")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = ["-O3", f"--offload-arch={ARCH}", "-std=c++17", "-fPIC", "-ffp-contract=on",
         "-fno-fast-math", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # matrix-core results in ordinary VGPRs (no accumulator-register copies)
         "-mllvm", "-amdgpu-mfma-vgpr-form",
         "-Wall", "-Wno-unused-function", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}"]


def _compile(src, verbose, out, more):
    obj = os.path.join(out, os.path.basename(src) + ".o")
    cmd = [HIPCC] + FLAGS + more + ["-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "warning: unknown target feature"
    err = "\n".join(l for l in (r.stderr or "").splitlines() if noise not in l and l.strip())
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if verbose and err:
        print(err, flush=True)
    return obj


def build(verbose=False, count_ends=False):
    """Compiles every csrc/*.hip for gfx950 and links libmclya.so (always).
    count_ends: libmclya_ends.so instead, whose tallies also hold the crossings
    that were counted without a step (as scatterings)."""
    lib, out = (LIB_ENDS, OBJ + "_ends") if count_ends else (LIB, OBJ)
    more = ["-DMCLYA_COUNT_ENDS"] if count_ends else []
    os.makedirs(out, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose, out, more), srcs))
    tmp = lib + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, lib)
    return lib


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv, count_ends="--count-ends" in sys.argv))
