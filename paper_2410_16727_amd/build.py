"""Build ``libdsopt.so`` (gfx950) in-tree with hipcc."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdsopt.so")
SOURCES = ["dsopt_kernels.hip", "dsopt_optimize_ext.hip", "dsopt_cost.hip", "dsopt_scene.hip",
           "dsopt_noalloc.hip", "dsopt_host.cpp", "dsopt_serve.cpp"]
ARCH = os.environ.get("DSOPT_ARCH", "gfx950")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC",
    f"--offload-arch={ARCH}",
    # packed FP32 instructions are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fno-gpu-rdc",
]


def build(verbose: bool = False, out: str = LIB, defines=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = out + ".tmp"

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("hipcc failed")

    flags = [*HIPCC_FLAGS, *[f"-D{d}" for d in defines], "-I", os.path.join(ROOT, "include"),
             "-I", CSRC]
    with tempfile.TemporaryDirectory() as d:
        # one object per source, side by side (the kernels' take minutes)
        objs = [os.path.join(d, s + ".o") for s in SOURCES]
        with ThreadPoolExecutor(max_workers=4) as ex:
            list(ex.map(lambda so: run([hipcc, *flags, "-c", os.path.join(CSRC, so[0]), "-o", so[1]]),
                        zip(SOURCES, objs)))
        run([hipcc, "-shared", f"--offload-arch={ARCH}", *objs, "-o", tmp])
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
