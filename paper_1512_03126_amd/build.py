"""Builds librdos.so in-tree for gfx950 with hipcc.

Floating point: -ffp-contract=off and no fast-math, so the FP64 expressions of
the kernels are evaluated exactly as written.  Packed-FP32 instructions are
disabled (-packed-fp32-ops).
"""
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librdos.so")
SOURCES = ["rdos_kernels.hip", "rdos_resident.hip", "rdos_sparse.hip", "rdos_api.cpp", "rdos_engine.cpp", "rdos_static.hip", "rdos_probes.hip"]
# Flags of single sources.  The step kernels' many 64-bit constants, hoisted
# out of the period loop, overflow the scalar registers into vector lanes: on
# the resident kernel 345 lane reads against 195 (abc, 384,000 tets: 10.05
# against 9.65 us per period).
SOURCE_FLAGS = {f: ["-mllvm", "-disable-machine-licm"] for f in ("rdos_resident.hip", "rdos_sparse.hip")}
ARCH = os.environ.get("RDOS_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def flags():
    return [
        "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
        "-ffp-contract=off", "-fno-fast-math",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-Wall", "-Wno-unused-result", "-pthread",
    ]


def build(verbose: bool = False) -> str:
    cc = hipcc()
    objs = []
    for src in SOURCES:
        path = os.path.join(CSRC, src)
        if not os.path.exists(path):
            continue
        obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
        lang = ["-x", "hip"]
        cmd = [cc, *flags(), *SOURCE_FLAGS.get(src, []), *lang, "-c", path, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [cc, *flags(), "-shared", "-o", tmp, *objs, "-pthread"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
