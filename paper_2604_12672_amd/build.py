"""Build the HIP library libmhd.so for gfx950 (in-tree).

hipcc compiles the kernels and the C-ABI host code, file by file in parallel,
and links them to one shared library.
Floating-point contraction is limited to single expressions
(-ffp-contract=on) so that a value recomputed by two blocks from the same
inputs rounds identically; packed FP32 instructions are disabled.
"""
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmhd.so")
SOURCES = ["mhd_api.hip", "mhd_kernels.hip", "mhd_diffusion.hip", "mhd_flatten.hip",
           "mhd_species.hip", "mhd_mathcheck.hip", "mhd_noalloc.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -amdgpu-mfma-vgpr-form: the matrix instructions of the guess network
# write their results to ordinary VGPRs, so the vector work that packs them
# for the next layer reads them directly instead of copying each value out
# of the accumulation registers first (the kernels without matrix
# instructions are unaffected).
# -amdgpu-sched-strategy=max-ilp: with the default strategy the FP64 stage
# kernel of the ideal gas without optional features (three waves per SIMD, 168
# registers) spills 22 registers and waits for every load in flight at each
# reload; with this one it fits 164 (256^3 stratified box, three steps: 14.8 ->
# 13.1 ms).  The other kernels of that file run as fast with either; the species
# and diffusion kernels lose 18 and 3 % with it, so the other files take the
# default.
STAGE_SCHED = ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]
STAGE_FILE = "mhd_kernels.hip"
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
    "-ffp-contract=on", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-result",
] + STAGE_SCHED


def flags_of(source: str) -> list:
    """Compile flags of one source file."""
    return FLAGS if source == STAGE_FILE else FLAGS[:-len(STAGE_SCHED)]


def build(verbose: bool = False, extra=None) -> str:
    extra = list(extra or [])
    with tempfile.TemporaryDirectory() as tmp:
        jobs, objs = [], []
        for s in SOURCES:
            objs.append(os.path.join(tmp, s + ".o"))
            cmd = ([HIPCC] + [f for f in flags_of(s) if f != "-shared"] + extra +
                   ["-c", os.path.join(CSRC, s), "-o", objs[-1]])
            if verbose:
                print(" ".join(cmd), flush=True)
            jobs.append((cmd, subprocess.Popen(cmd)))
        for cmd, job in jobs:
            if job.wait() != 0:
                for _, other in jobs:
                    other.wait()
                raise subprocess.CalledProcessError(job.returncode, cmd)
        link = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950"] + objs + ["-o", LIB + ".tmp"]
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.run(link, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
