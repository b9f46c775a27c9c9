"""Build libsppo.so in-tree with hipcc for gfx950.

Every HIP source under csrc/ is compiled to an object in csrc/../_build and
linked into paper_2503_10377_amd/libsppo.so.  Always recompiles (the caller
asked for a build).  Run as ``python -m paper_2503_10377_amd.build``.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libsppo.so")
ARCH = "gfx950"

# -packed-fp32-ops off: keep the compiler from forming v_pk_{add,mul,fma}_f32
# (the host pass warns that it does not know the feature; harmless).
COMMON = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE, "-I", CSRC, "-Wall", "-Wno-unused-function",
]

# Per-source extra flags.  The attention and GEMM kernels keep their MFMA
# results in arch VGPRs (the softmax reads S and dP with VALU ops, which would
# otherwise copy them out of AGPRs one register at a time); the compiler then
# places read-only MFMA operands (K/V or Q/dO fragments) in AGPRs.
EXTRA = {
    "attn_f32.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "gemm_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "attn_fwd_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "attn_bwd_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "attn_fwd_bf16_mfma32.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "attn_bwd_bf16_mfma32.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
}


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (need ROCm)")


def sources() -> list[str]:
    names = sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))
    return [os.path.join(CSRC, f) for f in names]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    cmd = [hipcc()] + COMMON + EXTRA.get(os.path.basename(src), []) + lang + ["-c", src, "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
