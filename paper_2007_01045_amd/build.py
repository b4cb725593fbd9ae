"""Build step: compile the HIP sources in csrc/ for gfx950 and link
libdapple_stage.so next to this file.  `python -m paper_2007_01045_amd.build`."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdapple_stage.so")
SOURCES = ["gemm_nn.hip", "gemm_nt.hip", "gemm_nn_pack.hip", "gemm_nt_pack.hip", "gemm_tn.hip", "gemm_tn_pack.hip", "gemm_tt.hip",
           "gemm_tt_pack.hip", "gemm_wgrad.hip", "gemm.hip", "gemm_f32.hip", "attention.hip", "attention_f32.hip",
           "rowops.hip", "embed_head.hip", "optimizer.hip", "stage.hip", "pipeline.hip", "kernel_api.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-result", "-Wno-inline-asm",
         # keep the compiler from forming packed-fp32 instructions
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # a kernel's first arguments arrive in scalar registers with the wave, instead of by a load from memory that everything
         # else waits for: kernels with arguments of their own (LayerNorm, sums, copies), not those with one structure (products,
         # attention).  An option of the compiler's back end; where the firmware lacks it, a kernel loads its arguments itself.
         # Three runs each in turn, us per iteration: 2 layers of 256 with 256 rows 264.5 -> 262.5 (spread 0.1%), 6 of 1024 with
         # 512 rows 1209 -> 1205 (0.2%), 4 of 768 with 600 rows 1904 -> 1896 (0.4%); large ones unchanged.
         "-mllvm", "-amdgpu-kernarg-preload-count=16"]


def _hipcc() -> str:
    for c in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.isabs(c) and os.path.exists(c):
            return c
    return "hipcc"


def _run(cmd):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops' is not a recognized feature" not in l)
    if p.returncode != 0:
        raise RuntimeError("command failed: " + " ".join(cmd) + "\n" + out)
    return out


def build(verbose: bool = False) -> str:
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    hipcc = _hipcc()
    objs = [os.path.join(bdir, s.replace(".hip", ".o")) for s in SOURCES]

    def compile_one(i):
        return _run([hipcc, *FLAGS, "-c", os.path.join(CSRC, SOURCES[i]), "-o", objs[i]])

    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        for out in ex.map(compile_one, range(len(SOURCES))):
            if verbose and out.strip():
                print(out)
    out = _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    if verbose and out.strip():
        print(out)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
