"""Builds libcodecsight.so (gfx950) in-tree with hipcc.  `python -m paper_2604_06036_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcodecsight.so")
SOURCES = ["library.hip", "calibrate.hip", "project_blocks.hip", "residual_proxy.hip", "score_compact.hip", "plan_refresh.hip", "kv_rerotate.hip", "window_attn.hip"]

# Packed-fp32 VALU forms are switched off for device code (scalar fp32 code generation only).  Matrix instructions keep
# their results in the vector registers unless the source says otherwise: the persistent attention kernel fills the
# accumulation registers with what it names itself, and its scores are read by vector instructions.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    "-Wno-unused-command-line-argument",
]


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                    if "packed-fp32-ops" not in l and l.strip())
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out:
        print(out)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
