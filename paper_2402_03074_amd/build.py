"""Build libhwenou.so in-tree with hipcc for gfx950.

Every HIP translation unit is compiled with packed FP32 instructions disabled
(`-Xclang -target-feature -Xclang -packed-fp32-ops`).
"""
import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libhwenou.so")
SOURCES = ["hwenou_api.hip", "stage1d.hip", "step1d.hip", "stage2d.hip", "pair2d.hip",
           "aux.hip", "noalloc.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = os.environ.get("HWENOU_ARCH", "gfx950")

FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unused-command-line-argument"]


# Per-file flags.  The 2D stage kernel runs one wave per SIMD, so nothing
# hides its latencies but its own instruction order; LLVM's iterative ILP
# scheduler orders it better than the default (mixed form: 4% per stage).
# That scheduler fails on the 1D kernels; the max-ILP one orders them 2%
# better than the default on a batch of 512 grids.
SOURCE_FLAGS = {"stage2d.hip": ["-mllvm", "-amdgpu-sched-strategy=iterative-ilp"],
                "stage1d.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"],
                "step1d.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"],
                "pair2d.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]}


def _compile(src, verbose, extra):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    base = [HIPCC] + FLAGS + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
    cmd = base[:1] + SOURCE_FLAGS.get(src, []) + base[1:]
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0 and SOURCE_FLAGS.get(src):
        # the scheduler is experimental: fall back to the default one (same
        # results, somewhat slower) rather than fail the build
        print(f"warning: {src} failed with {' '.join(SOURCE_FLAGS[src])}; "
              "building it with the default scheduler", file=sys.stderr)
        r = subprocess.run(base, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    out = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l
                    and "is not a recognized feature" not in l)
    return obj, out


def build(verbose=False, resource_usage=False):
    os.makedirs(BUILD, exist_ok=True)
    extra = ["-Rpass-analysis=kernel-resource-usage"] if resource_usage else []
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        results = list(ex.map(lambda s: _compile(s, verbose, extra), SOURCES))
    objs = [r[0] for r in results]
    logs = [r[1] for r in results if r[1].strip()]
    if logs and (verbose or resource_usage):
        print("\n".join(logs), file=sys.stderr)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}"] + objs + ["-o", tmp]
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv, resource_usage="--usage" in sys.argv)
    print(LIB)
