"""Builds libregenvc_attn.so for gfx950 with hipcc (in-tree, no JIT cache).

Run as ``python -m paper_2607_28144_amd.build``; it compiles every time it is
called.  Packed-fp32 VALU instructions are switched off for all device code.
"""
import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
REPO_DIR = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_NAME = "libregenvc_attn.so"
LIB_PATH = os.path.join(PKG_DIR, LIB_NAME)
SOURCES = ["api.cpp", "attn_fwd.hip", "lse_merge.hip", "norm_rope.hip", "dit_api.cpp", "dit.hip", "vae_api.cpp",
           "vae.hip"]
ARCH = "gfx950"
# MFMA results in VGPRs: the score tiles feed VALU softmax code directly, and
# read-only operands may then live in AGPRs.  Not for the tile kernels of the
# linear layers, whose accumulators fill the AGPRs.
VGPR_FORM = {"attn_fwd.hip"}


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def build(verbose: bool = False) -> str:
    """Compile the shared library; returns its path.  Raises on failure."""
    out_tmp = LIB_PATH + ".tmp"
    flags = [
        f"--offload-arch={ARCH}",
        "-O3",
        "-std=c++17",
        "-fPIC",
        "-Wall",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", os.path.join(REPO_DIR, "include"),
        "-I", CSRC,
    ]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        # the host pass does not know the packed-fp32 feature: that warning is harmless
        msgs = [ln for ln in (res.stdout + res.stderr).splitlines() if "packed-fp32-ops" not in ln]
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + "\n".join(msgs))
        remarks = [ln for ln in msgs if "kernel-resource-usage" in ln]
        msgs = [ln for ln in msgs if "kernel-resource-usage" not in ln and not re.match(r"^\s*\d*\s*\||^\s*\^", ln)]
        if verbose and msgs:
            print("\n".join(msgs), flush=True)
        return remarks

    def compile_one(name, obj):
        extra = ["-mllvm", "-amdgpu-mfma-vgpr-form"] if name in VGPR_FORM else []
        kernel = ""
        for ln in run([hipcc()] + flags + extra + ["-Rpass-analysis=kernel-resource-usage", "-c", "-o", obj,
                                                   os.path.join(CSRC, name)]):
            if "Function Name:" in ln:
                kernel = ln
            # tiles whose MFMAs are instructions of their own: no spill may touch their accumulators
            elif "Shape4" in kernel and "Spill" in ln and not re.search(r"Spill: 0\b", ln):
                raise RuntimeError(f"{name}: a four-wave tile kernel spills: {kernel} {ln}")

    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        with ThreadPoolExecutor(max_workers=4) as pool:
            list(pool.map(compile_one, SOURCES, objs))
        run([hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", out_tmp] + objs)
    os.replace(out_tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
