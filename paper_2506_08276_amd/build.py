"""Builds libleann.so (gfx950) in-tree with hipcc."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libleann.so")
SOURCES = ["api.hip", "encoder.hip", "pq.hip", "search.hip", "build.hip", "peak.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument"]
# Kernel arguments come in scalar registers with the dispatch, as many as there is room for: read from memory, they are the first
# link of every kernel's chain of latencies.  Embedding one chunk, 87 dependent launches, took 424 us without, 401 with it.  For the files
# with such chains; arguments in a struct stay in memory, as those of a launch that nothing runs ahead of should (adc_direct_kernel).
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]
FLAGS_OF = {"encoder.hip": PRELOAD, "pq.hip": PRELOAD}


def build_library(verbose=False):
    """Compile every HIP source and link the shared library; returns its path."""
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
        cmd = ["hipcc", *FLAGS, *FLAGS_OF.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
