"""Build the simulator's shared library in-tree for gfx950.

    python -m paper_2605_15098_amd.build

Produces ``paper_2605_15098_amd/libsvmi.so`` from ``csrc/`` with hipcc. The
packed-FP32 target feature is switched off for all device code.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsvmi.so")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HIPCC = os.environ.get("HIPCC", os.path.join(ROCM, "bin", "hipcc"))

SOURCES = ["block.hip", "batch.hip", "kernels.hip", "readout.hip", "mlp.hip", "api.cpp", "plan.cpp", "jit.cpp", "qasm.cpp"]
# headers embedded as text for the pass kernels compiled at run time
JIT_HEADERS = [("kJitAbiH", "k2_abi.h"), ("kJitDeviceH", "k2_device.h")]


def write_jit_sources() -> None:
    out = ["// generated by build.py from the headers below; do not edit"]
    for var, name in JIT_HEADERS:
        with open(os.path.join(CSRC, name)) as fh:
            text = fh.read()
        assert ")SVJIT" not in text
        out.append(f'static const char *const {var} = R"SVJIT({text})SVJIT";')
    dst = os.path.join(CSRC, "jit_src.inc")
    new = "\n".join(out) + "\n"
    if not os.path.exists(dst) or open(dst).read() != new:
        with open(dst, "w") as fh:
            fh.write(new)
# Device code: packed FP32 off; no implicit contraction into FMA (every fused
# multiply-add in the kernels is an explicit fma), so a gate sequence rounds
# the same whether its gates run as separate kernels, interpreted ops or one
# generated pass.
DEVICE_FLAGS = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=off"]


# The interpreters' op loop branches only on uniform values. Structurizing it
# merges the paths of all handlers through copies of the thread's whole register
# tile, twice an op (289 vector instructions per amplitude and pass of the
# batched phase estimations); uniform regions are left as they are.
INTERP_FLAGS = ["-mllvm", "-structurizecfg-skip-uniform-regions"]
INTERP_SOURCES = ("block.hip", "batch.hip")


def build(verbose: bool = False) -> str:
    write_jit_sources()
    objs, cmds = [], []
    for src in SOURCES:
        path = os.path.join(CSRC, src)
        obj = os.path.join(CSRC, src + ".o")
        cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-c", path, "-o", obj,
               "-Wall", "-Wno-unused-function"]
        if src.endswith(".hip"):
            cmd += DEVICE_FLAGS + (INTERP_FLAGS if src in INTERP_SOURCES else [])
        else:
            # host-only translation units: plain g++ against the HIP runtime headers
            cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-c", path, "-o", obj, "-Wall",
                   "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include"]
        if verbose:
            print(" ".join(cmd), flush=True)
        cmds.append(cmd)
        objs.append(obj)
    # block.hip and batch.hip take minutes (every register tile of the interpreter), the rest seconds
    with ThreadPoolExecutor(5) as pool:
        list(pool.map(lambda c: subprocess.run(c, check=True), cmds))
    tmp = LIB + f".tmp{os.getpid()}"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs + \
        [f"-L{ROCM}/lib", "-lhiprtc", f"-Wl,-rpath,{ROCM}/lib"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
