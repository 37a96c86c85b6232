"""Build libmorea.so for gfx950 with hipcc (in-tree, next to this file)."""
import concurrent.futures
import glob
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libmorea.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # packed FP32 instructions are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]
# Schedule for instruction-level parallelism where long straight-line samples
# bound the kernel: 128x128x96, 512 candidates 8.39 -> 8.28 ms, 32,768 partial
# evaluations 33.96 -> 33.14 ms, Sobol points of 128 candidates 2.82 -> 2.74 ms.
# Training loses by it (65,536 rows, calls one by one: 35.4 -> 37.1 us), the
# others do not change.
ILP = ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]
FILE_FLAGS = {"morea_eval.hip": ILP, "morea_sobol.hip": ILP}


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def build(verbose: bool = False) -> str:
    """Compile every HIP source into libmorea.so (always rebuilds)."""
    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)

    def compile_one(src, obj):
        run([HIPCC] + FLAGS + FILE_FLAGS.get(os.path.basename(src), []) +
            ["-I", os.path.join(HERE, "..", "include"), "-c", src, "-o", obj])

    with tempfile.TemporaryDirectory() as d:
        objs = [os.path.join(d, os.path.basename(src) + ".o") for src in sources()]
        with concurrent.futures.ThreadPoolExecutor(max_workers=min(4, os.cpu_count() or 1)) as pool:
            list(pool.map(compile_one, sources(), objs))
        tmp = LIB + ".tmp%d" % os.getpid()
        run([HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
