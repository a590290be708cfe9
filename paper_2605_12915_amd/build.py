"""Build libaf.so (HIP, gfx950) in-tree.

    python -m paper_2605_12915_amd.build
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libaf.so")
ARCH = os.environ.get("AF_OFFLOAD_ARCH", "gfx950")

HIPCC = "/opt/rocm/bin/hipcc"
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-munsafe-fp-atomics", f"-I{CSRC}", f"-I{INCLUDE}",
]
# FP contraction: free (across statements) for the FP64 kernels; within source
# expressions only for the FP32 step kernels, which must round identically.
CONTRACT_ON = {"af_fused_f32.hip", "af_fused_f32_small.hip", "af_batch.hip"}
# Files whose LDS reads stay single: a ds_read2_b64 holds the LDS for 8.2 cycles, two
# ds_read_b64 for 4.7 (16 waves per CU).  The FP32 31x10 and batch kernels are the faster with
# paired reads, which cost them no LDS cycles and save issue slots.
SINGLE_READS = {"af_adjoint.hip", "af_fused.hip", "af_fused_f32_small.hip"}


# Backend options for the device code only (a plain -mllvm would also reach the host
# compile, whose target does not know them): the GCN max-ILP machine scheduler, 1.5-3%
# faster on the step, FP32 and adjoint kernels than the default.  The device pass writes
# the offload bundle that the host pass embeds.
DEVICE_ONLY = ["-mllvm", "-misched=gcn-max-ilp"]
UNPAIRED = ["-Xclang", "-target-feature", "-Xclang", "-load-store-opt", "-mllvm", "-amdgpu-load-store-vectorizer=0"]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    dev = os.path.join(OBJ, os.path.basename(src) + ".hipfb")
    contract = "-ffp-contract=on" if os.path.basename(src) in CONTRACT_ON else "-ffp-contract=fast"
    reads = UNPAIRED if os.path.basename(src) in SINGLE_READS else []
    cmds = [[HIPCC, *FLAGS, contract, "--cuda-device-only", *DEVICE_ONLY, *reads, "-c", src, "-o", dev],
            [HIPCC, *FLAGS, contract, "--cuda-host-only", "-Xclang", "-fcuda-include-gpubinary", "-Xclang", dev,
             "-c", src, "-o", obj]]
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    return obj


def build(verbose: bool = False) -> str:
    subprocess.run([sys.executable, os.path.join(CSRC, "gen_blocks.py")], check=True)
    subprocess.run([sys.executable, os.path.join(CSRC, "gen_gauss.py")], check=True)
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
