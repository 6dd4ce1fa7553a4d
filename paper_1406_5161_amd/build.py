"""Build libsvmhip.so (HIP, gfx950) in-tree with hipcc."""
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libsvmhip.so")
SOURCES = ["svm_step.hip", "svm_reg_dense.hip", "svm_reg_bits.hip", "svm_batch.hip", "svm_kernels.hip", "svm_ksum_ht.hip", "svm_shared.hip", "svm_noalloc.hip", "svm_host.cpp", "svm_serve.cpp", "svm_tune.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no hand-written or compiler-generated packed FP32 arithmetic
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def build(verbose: bool = False) -> str:
    """Compile every source (each on its own, a few at a time) and link the library."""
    tmp = LIB + ".tmp%d" % os.getpid()
    work = tempfile.mkdtemp(prefix="svmhip_build_")

    def compile_one(name):
        obj = os.path.join(work, name + ".o")
        cmd = [HIPCC] + FLAGS + ["-x", "hip", "-c", "-o", obj, os.path.join(CSRC, name)]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    try:
        with ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            objs = list(pool.map(compile_one, SOURCES))
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
    finally:
        shutil.rmtree(work, ignore_errors=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
