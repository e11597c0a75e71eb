"""Build libddpinn.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libddpinn.so")
BUILD = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
# Packed FP32 instructions are disabled for every device compile.
DEVICE_FLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC",
                "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                "-munsafe-fp-atomics"]
HOST_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-result"]

# (source, defines): the network kernels are compiled once per dimension (and
# activation), in parallel
SOURCES = ([("ddpinn_step.hip", [f"-DDDP_DIM={d}", f"-DDDP_ACT={a}"]) for d in (3, 2) for a in (1, 0)] +
           [("ddpinn_query.hip", [f"-DDDP_DIM={d}"]) for d in (2, 3)] +
           [("ddpinn_wide.hip", []), ("ddpinn_kernels.hip", []), ("ddpinn_api.cpp", [])])


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("build failed: " + " ".join(cmd) + "\n" + out)
    return out


def build(verbose: bool = False) -> str:
    """Compile every source and link libddpinn.so (always rebuilds)."""
    os.makedirs(BUILD, exist_ok=True)
    def one(entry):
        src, defs = entry
        path = os.path.join(CSRC, src)
        obj = os.path.join(BUILD, src + "".join(defs).replace("-D", ".") + ".o")
        if src.endswith(".hip"):
            cmd = [HIPCC, *DEVICE_FLAGS, *defs, "-I", INCLUDE, "-I", CSRC, "-c", path, "-o", obj]
        else:
            cmd = [HIPCC, "-x", "c++", *HOST_FLAGS, "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", INCLUDE,
                   "-I", CSRC, "-c", path, "-o", obj]
        out = _run(cmd)
        if verbose and out.strip():
            print(out)
        return obj

    with ThreadPoolExecutor(max_workers=8) as pool:   # the compilers run as child processes
        objs = list(pool.map(one, SOURCES))
    tmp = LIB + ".tmp"
    _run([HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
