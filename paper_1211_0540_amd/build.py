"""Build libbz.so (HIP, gfx950) in-tree.

Every HIP source is compiled with packed FP32 instructions disabled
(-packed-fp32-ops); hipcc's host pass warns that it does not know the
feature, which is harmless.
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbz.so")
# (source, object, defines), longest first; the convolution kernels compile in four units
UNITS = [("bz_conv.hip", f"bz_conv{u}.o", [f"-DBZ_CONV_UNIT={u}"]) for u in (0, 2, 3, 1)]
UNITS += [(f"bz_{n}.hip", f"bz_{n}.o", []) for n in ("dft", "runtime", "surrogate", "misc", "mlp", "transport")]
ARCH = os.environ.get("BZ_OFFLOAD_ARCH", "gfx950")


def hipcc_flags():
    return ["-O3", "-std=c++20", f"--offload-arch={ARCH}", "-fPIC",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wno-unused-command-line-argument", "-I", os.path.join(HERE, "..", "include")]


def build(verbose: bool = False, jobs: int = 10) -> str:
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src, name, defs in UNITS:
        obj = os.path.join(HERE, "_build", name)
        cmd = ["hipcc", *hipcc_flags(), *defs, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((subprocess.Popen(cmd), src))
        objs.append(obj)
        while len([p for p, _ in procs if p.poll() is None]) >= jobs:
            procs[[p.poll() is None for p, _ in procs].index(True)][0].wait()
    for p, src in procs:
        if p.wait() != 0:
            raise RuntimeError(f"hipcc failed on {src}")
    cmd = ["hipcc", f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
