"""Builds the FlashOptim HIP library for gfx950 in-tree: paper_2602_23349_amd/libflashoptim.so."""
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libflashoptim.so")
SOURCES = [os.path.join(CSRC, "flashoptim_kernels.hip"), os.path.join(CSRC, "flashoptim_api.hip")]
HEADERS = [os.path.join(CSRC, "flashoptim_device.h"), os.path.join(CSRC, "flashoptim_launch.h"),
           os.path.join(ROOT, "include", "flashoptim.h")]

# Exact arithmetic is part of the contract: no FMA contraction, IEEE division and square root,
# subnormals kept.  Packed FP32 instructions are disabled.  The command processor loads a kernel's first arguments into
# registers before its wavefronts start (up to 14 words), instead of every wavefront by a load that it waits for.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-gpu-flush-denormals-to-zero",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=16",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(p) > t for p in SOURCES + HEADERS + [os.path.abspath(__file__)])     # (this file: the flags)


def build(force: bool = True) -> str:
    if not force and not stale():
        return LIB
    cmd = [hipcc()] + FLAGS + SOURCES + ["-o", LIB]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass warns that it does not know the packed-fp32-ops feature: harmless
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if out.strip():
        print(out, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build())
