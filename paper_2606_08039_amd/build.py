"""Build libmd.so (HIP for gfx950) in-tree with hipcc.

``python -m paper_2606_08039_amd.build`` or ``build.build()``.  Every call
compiles; nothing is cached.  All device code is compiled with packed FP32
instructions disabled.
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmd.so")

HIP_SOURCES = ["md_mlp.hip", "md_surrogate.hip"]
# one object per action type (-DMD_ACT=0..4)
ACT_SOURCES = ["md_step.hip", "md_step_dr.hip", "md_step_wind.hip", "md_rk4.hip"]
CPP_SOURCES = ["md_api.cpp", "md_tune.cpp"]

ARCH = "gfx950"
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          "-I", os.path.join(ROOT, "include"), "-I", CSRC]
DEVICE = ["--offload-arch=" + ARCH, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-munsafe-fp-atomics"]
# per-source options: the surrogate step keeps its MFMA accumulators in
# ordinary VGPRs, so that the SiLU epilogue reads them without a copy out of
# the accumulation registers
EXTRA = {"md_surrogate.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)


def objects():
    """(source, object, compiler options) of everything in libmd.so."""
    bdir = os.path.join(HERE, "_build")
    jobs = [(src, "%s.%d.o" % (src, act), ["-x", "hip", "-DMD_ACT=%d" % act]) for src in ACT_SOURCES for act in range(5)]
    jobs += [(src, src + ".o", ["-x", "hip"] + EXTRA.get(src, [])) for src in HIP_SOURCES]
    jobs += [(src, src + ".o", []) for src in CPP_SOURCES]
    return [(src, os.path.join(bdir, obj), opt) for src, obj, opt in jobs]


def build(verbose=False, jobs=8):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)

    def compile_one(job):
        src, obj, opt = job
        _run([hipcc] + opt + ["-c"] + COMMON + DEVICE + [os.path.join(CSRC, src), "-o", obj], verbose)

    todo = objects()
    with ThreadPoolExecutor(jobs) as pool:
        for f in [pool.submit(compile_one, j) for j in todo]:
            f.result()
    tmp = LIB + ".tmp%d" % os.getpid()
    _run([hipcc, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", tmp] + [obj for _, obj, _ in todo], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
