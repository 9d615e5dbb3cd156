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
# Sources with tiles whose MFMAs are instructions of their own (inline
# assembly, around which the compiler places no wait states): their assembly is
# checked (check_tile_kernels).
CHECKED = {"dit.hip", "vae.hip"}


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def check_tile_kernels(name: str, asm: str) -> int:
    """Refuses device assembly in which a tile kernel with one wave per SIMD
    spills, or in which an instruction other than an MFMA touches an
    accumulator (AGPR) less than 20 wait states after an MFMA or 4 before one,
    on any path: the compiler places none around its inline MFMAs.  Returns
    the number of kernels checked; none is an error."""
    def fail(kernel, what):
        raise RuntimeError(f"{name}: {what}: {kernel}")

    one_wave = re.compile(r"Shape4I(?:Li\d+E){3}Li1EE")
    meta = {}
    for entry in re.split(r"(?m)^  - (?=\.\w+:)", asm)[1:]:
        keys = dict(re.findall(r"(?m)^\s*(\.\w+):\s+(\S+)\s*$", entry))
        if ".vgpr_spill_count" in keys:
            meta[keys[".name"]] = keys
    count = 0
    for text in re.split(r"(?m)^(?=_Z\w+:)", asm)[1:]:
        kernel = text.split(":", 1)[0]
        code = [ln.split(";")[0].strip() for ln in text.split(".Lfunc_end", 1)[0].splitlines()[1:]]
        code = [ln for ln in code if ln.startswith(".LBB") or ln and not ln.startswith(".")]
        mfma = [ln.startswith("v_mfma") for ln in code]
        if not one_wave.search(kernel) or not any(mfma):
            continue
        if any(meta.get(kernel, {}).get(k) != "0" for k in (".vgpr_spill_count", ".sgpr_spill_count",
                                                            ".private_segment_fixed_size")):
            fail(kernel, "a tile kernel spills, or its resources are not listed")
        acc = [not m and re.search(r"\ba(?:\d|\[)", ln) is not None for m, ln in zip(mfma, code)]
        before = {}  # position -> positions that may run just before it
        labels = {ln[:-1]: i for i, ln in enumerate(code) if ln.endswith(":")}
        for i, ln in enumerate(code):
            op, _, target = ln.partition(" ")
            if target in labels:
                before.setdefault(labels[target], []).append(i)
            if op not in ("s_branch", "s_endpgm") and i + 1 < len(code):
                before.setdefault(i + 1, []).append(i)

        def within(start, states, hit):
            """A position of `hit` reached backwards from start over less than `states` wait states."""
            todo, seen = [(p, states) for p in before.get(start, [])], {}
            while todo:
                i, left = todo.pop()
                if hit[i]:
                    return True
                left -= 0 if code[i].endswith(":") else int(code[i].split()[1]) + 1 if code[i].startswith("s_nop") else 1
                if left > 0 and seen.get(i, 0) < left:
                    seen[i] = left
                    todo += [(p, left) for p in before.get(i, [])]
            return False
        if any(within(i, 20, mfma) for i in range(len(code)) if acc[i]) or \
                any(within(i, 4, acc) for i in range(len(code)) if mfma[i]):
            fail(kernel, "an accumulator is touched beside the MFMAs of a tile kernel")
        count += 1
    if count == 0:
        raise RuntimeError(f"{name}: no tile kernel found to check")
    return count


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
        if verbose and msgs:
            print("\n".join(msgs), flush=True)

    def compile_one(name, obj):
        extra = ["-mllvm", "-amdgpu-mfma-vgpr-form"] if name in VGPR_FORM else []
        cmd = [hipcc()] + flags + extra
        if obj.endswith(".s"):
            run(cmd + ["--cuda-device-only", "-S", "-o", obj, os.path.join(CSRC, name)])
            with open(obj) as f:
                check_tile_kernels(name, f.read())
        else:
            run(cmd + ["-c", "-o", obj, os.path.join(CSRC, name)])

    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        with ThreadPoolExecutor(max_workers=6) as pool:
            listings = [os.path.join(tmp, s + ".s") for s in sorted(CHECKED)]
            list(pool.map(compile_one, SOURCES + sorted(CHECKED), objs + listings))
        run([hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", out_tmp] + objs)
    os.replace(out_tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
