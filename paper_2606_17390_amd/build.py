"""Build libfem.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2606_17390_amd.build [--verbose]

Each .hip translation unit is compiled to an object in parallel, then linked
into paper_2606_17390_amd/libfem.so.
"""
import argparse
import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfem.so")
SOURCES = ["api.hip", "pattern.hip", "forward.hip", "vjp.hip", "solver.hip", "amg.hip", "adjoint.hip"]
ARCH = os.environ.get("FEM_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # packed FP32 instructions disabled
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # FP32 division and square root by the hardware reciprocal / square-root
    # approximations (about 1 ulp) instead of correctly rounded sequences; only
    # the FP32 part of the mixed-precision path uses them
    "-fno-hip-fp32-correctly-rounded-divide-sqrt",
    "-munsafe-fp-atomics",
    "-Wall", "-Wno-unused-function",
]

# The element kernels loop over tiles and use some 60 floating-point constants.
# Hoisted out of the loop these take up to 70 registers, which is what decides
# how many waves a SIMD holds; they are rebuilt where they are used instead.
SOURCE_FLAGS = {
    "forward.hip": ["-mllvm", "-disable-machine-licm"],
    "vjp.hip": ["-mllvm", "-disable-machine-licm"],
}


def _hipcc():
    for c in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.isabs(c) and os.path.exists(c):
            return c
    return "hipcc"


def compile_one(src, extra, verbose):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *FLAGS, *SOURCE_FLAGS.get(src, []), *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj, r.stderr


def build(verbose=False, extra=()):
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(6, len(SOURCES))) as ex:
        results = list(ex.map(lambda s: compile_one(s, list(extra), verbose), SOURCES))
    objs = [o for o, _ in results]
    for _, err in results:
        if verbose and err.strip():
            print(err)
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--verbose", action="store_true")
    ap.add_argument("--resource-usage", action="store_true",
                    help="print per-kernel register / LDS / scratch usage")
    args = ap.parse_args()
    extra = ["-Rpass-analysis=kernel-resource-usage"] if args.resource_usage else []
    print(build(args.verbose or args.resource_usage, extra))


if __name__ == "__main__":
    sys.exit(main())
