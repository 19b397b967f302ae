"""Builds the engine's shared library (libn2v.so) for gfx950 with hipcc."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libn2v.so")
SOURCES = ["api.hip", "prims.hip", "rmat.hip", "graph.hip", "walk.hip", "tune.hip", "server.hip", "skipgram.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # keep packed FP32 instructions out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-result",
]
# The persistent walk kernel is held to 80 VGPRs (six wavefronts per SIMD;
# weighted 96, five).  The compiler hoists the hub path's lane constants out of
# the walk loop, where they push the lanes' walk state into scratch (86 spilled
# registers, weighted 166), stored and reloaded on every rejection move.
# Sinking them back leaves none (3).  When the flag came (one kernel of 96
# registers): ER-22 29.2 -> 24.2 ms, WeC-22 72.9 -> 67.7 ms, FN-Approx on Skew-5
# 172.6 -> 158.0 ms, weighted scale 20 278 -> 252 ms.  The Skip-gram kernel
# spills nothing and is 5% slower with it, so it is a flag of walk.hip alone.
SOURCE_FLAGS = {"walk.hip": ["-mllvm", "-sink-insts-to-avoid-spills=1"]}


def build(verbose: bool = False, jobs: int = 4) -> str:
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs, objs = [], []
    for src in SOURCES:
        path = os.path.join(CSRC, src)
        obj = os.path.join(objdir, src + ".o")
        objs.append(obj)
        cmd = [HIPCC] + FLAGS + SOURCE_FLAGS.get(src, []) + ["-c", path, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        if len([p for _, p in procs if p.poll() is None]) >= jobs:
            procs[-jobs][1].wait()
    failed = []
    for src, p in procs:
        out = p.communicate()[0].decode()
        if p.returncode != 0:
            failed.append((src, out))
        elif verbose and out.strip():
            print(out)
    if failed:
        msg = "\n".join(f"--- {s}\n{o}" for s, o in failed)
        raise RuntimeError("HIP build failed:\n" + msg)
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs + ["-lpthread"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
