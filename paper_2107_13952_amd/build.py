"""Compile the HIP library ``libeprl.so`` in-tree for gfx950 with hipcc."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libeprl.so")
SOURCES = ["sixj.hip", "assemble.hip", "ring.hip", "chain.hip", "contract.hip", "adjoint_ring.hip", "network.hip", "boosters.hip",
           "eprl_plan.cpp", "api.cpp"]

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # keep the compiler from emitting packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-result",
]


def build(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp"

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError("hipcc failed building libeprl.so")

    # One compilation per source, at most eight at a time, then the link.
    with tempfile.TemporaryDirectory() as objs, ThreadPoolExecutor(8) as pool:
        out = [os.path.join(objs, s + ".o") for s in SOURCES]
        list(pool.map(run, [[hipcc] + FLAGS + ["-c", "-o", o, os.path.join(CSRC, s)]
                            for s, o in zip(SOURCES, out)]))
        run([hipcc] + FLAGS + ["-shared", "-o", tmp] + out)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
