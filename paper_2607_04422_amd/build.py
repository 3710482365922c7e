"""Build libfp4root.so (HIP kernels + C ABI) for gfx950 with hipcc, in the package directory."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfp4root.so")
# sweeps of the device helpers over their ranges, loaded by tests only
SWEEPS = os.path.join(HERE, "libfp4root_sweeps.so")
SOURCES = ["quant.hip", "gemm_fp4.hip", "gemm_bf16.hip", "gemm_blaslt.cpp", "optim.hip", "api.cpp"]
# the update product of the BF16 comparison path is a hipBLASLt GEMM
LINK_LIBS = ["-L/opt/rocm/lib", "-lhipblaslt", "-Wl,-rpath,/opt/rocm/lib"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # bit-exact quantiser and epilogues: no FMA contraction, IEEE division
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    # never emit packed FP32 arithmetic
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]
# per-source extra flags: the exact NVFP4 product reads every MFMA result on the
# VALU, so its MFMA results live in VGPRs; the BF16 product keeps accumulators in AGPRs
SOURCE_FLAGS = {"gemm_fp4.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False, jobs: int = 3, extra_flags=(), out: str = LIB) -> str:
    """Compile every source for gfx950 and link the library (default libfp4root.so); returns its path."""
    objdir = os.path.join(HERE, "_build", os.path.basename(out) + ".d")
    os.makedirs(objdir, exist_ok=True)
    cc = hipcc()
    procs, objs = [], []
    for src in SOURCES:
        obj = os.path.join(objdir, src + ".o")
        objs.append(obj)
        cmd = [cc, *HIPCC_FLAGS, *SOURCE_FLAGS.get(src, []), *extra_flags, "-x", "hip", "-c",
               os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        if len(procs) >= jobs:
            _wait(procs.pop(0))
    while procs:
        _wait(procs.pop(0))
    tmp = out + ".tmp"
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, *LINK_LIBS, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stdout)
    os.replace(tmp, out)
    return out


def build_sweeps() -> str:
    """Compile probes/exact_math.hip (device helpers against the general operations)."""
    cmd = [hipcc(), *HIPCC_FLAGS, "-shared", "-x", "hip", os.path.join(HERE, "probes", "exact_math.hip"),
           "-o", SWEEPS + ".tmp"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed on probes/exact_math.hip:\n" + res.stdout)
    os.replace(SWEEPS + ".tmp", SWEEPS)
    return SWEEPS


def _wait(item):
    src, p = item
    out, _ = p.communicate()
    text = out.decode(errors="replace")
    if p.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{text}")
    errs = [ln for ln in text.splitlines() if "error" in ln.lower()]
    if errs:
        print(text, file=sys.stderr)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
    print(build_sweeps())
