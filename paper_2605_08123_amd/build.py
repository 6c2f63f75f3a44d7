"""Compile the HIP library for gfx950 in-tree (paper_2605_08123_amd/libsinkhorn_attn.so)."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libsinkhorn_attn.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA results straight into VGPRs (no accumulator-register copies before the VALU work)
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-I" + os.path.join(ROOT, "include"),
]
# Objects: the library, and the step kernel's instances by storage type and head dimension (most of it).  Compiled side by side.
UNITS = [("sinkhorn_attn", "sinkhorn_attn.hip", [])] + [
    (f"steps_{name}_{d}", "ska_step_launch.hip", [f"-DSKA_T={t}", f"-DSKA_D={d}", f"-DSKA_NAME=ska_launch_steps_{name}_{d}"])
    for name, t in (("bf16", "__bf16"), ("f32", "float")) for d in (64, 32, 128)]


def build_library(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

    def run(cmd):
        res = subprocess.run(cmd, capture_output=True, text=True)
        noise = "is not a recognized feature for this target"
        err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + err)
        if verbose and err.strip():
            print(err)

    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, name + ".o") for name, _, _ in UNITS]
        with ThreadPoolExecutor(max_workers=min(len(UNITS), os.cpu_count() or 1)) as pool:
            list(pool.map(lambda u: run([hipcc, *HIPCC_FLAGS, *u[0][2], "-c", "-o", u[1], os.path.join(CSRC, u[0][1])]), zip(UNITS, objects)))
        run([hipcc, "-shared", "-fPIC", "-o", LIB, *objects])
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
