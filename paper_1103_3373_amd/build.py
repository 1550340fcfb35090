"""Build libhydro.so (HIP, gfx950) in-tree with hipcc.

Every source under csrc/ is compiled for gfx950 only and linked into
paper_1103_3373_amd/libhydro.so.  Packed FP32 instructions are disabled
(-packed-fp32-ops) for the whole device code.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libhydro.so")
ARCH = os.environ.get("HYDRO_OFFLOAD_ARCH", "gfx950")

CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    "-Wno-unused-variable", "-Wno-unused-but-set-variable", "-Wno-unused-result", "-Wno-unused-value",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]
# Per-file additions.  The CTU kernels build with the AMDGPU scheduler's
# register-pressure trackers that follow the register allocator's own
# accounting.  256^3 box steps, us (FP32, PPM): default, trackers, max-ILP,
# max-memory-clause and iterative-minreg schedules:
#   CTU/HLLC            1226, 1122, 1262, 1270, 1277
#   CTU/Roe             1538, 1707, 1696, 1702, 1690
#   MHM/HLLC             845,  844,  836,  855,  965
#   MHM/HLLC + fluxes    869,  852,  869,  879,  995
#   MHM/Roe + fluxes     947,  911,  952,  950, 1075
#   VL/HLLC             1010,  964, 1002, 1013, 1167
EXTRA = {
    "fused_ctu_f32.hip": ["-mllvm", "-amdgpu-use-amdgpu-trackers=1"],
    # VL and MHM with the flux code take the trackers, MHM without it max-ILP,
    # the FP32 Roe CTU file (fused_ctu_f32_roe.hip) the default.
    "fused_muscl_f32.hip": ["-mllvm", "-amdgpu-use-amdgpu-trackers=1"],
    "fused_muscl_f32_mhm.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"],
    "fused_ctu_f64.hip": ["-mllvm", "-amdgpu-use-amdgpu-trackers=1"],
}


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = ["hipcc", *CFLAGS, *EXTRA.get(os.path.basename(src), []), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    # hipcc's host pass warns that it does not know the packed-fp32 feature.
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if err.strip():
        print(err, file=sys.stderr)
    return obj


def build(jobs: int | None = None) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    jobs = jobs or min(len(srcs), int(os.environ.get("MAX_JOBS", "8")))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    subprocess.check_call(["hipcc", f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
