"""Build the HIP library in-tree: paper_2604_05417_amd/libmetasd.so (gfx950 only)."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "metasd.hip")
DEPS = [SRC, os.path.join(HERE, "csrc", "kernels.h"), os.path.join(HERE, "csrc", "batch.h"), os.path.join(HERE, "csrc", "prefill.h"),
        os.path.join(HERE, "csrc", "gemm_tiles.h"), os.path.join(HERE, "csrc", "step.h"), os.path.join(HERE, "csrc", "attn.h"),
        os.path.join(HERE, "csrc", "attn_plan.h"),
        os.path.join(HERE, "csrc", "step_f32.h"), os.path.join(HERE, "csrc", "chain_f32.h"),
        os.path.join(HERE, "csrc", "chain_plan.h"),
        os.path.join(HERE, "..", "include", "metasd.h")]
LIB = os.path.join(HERE, "libmetasd.so")

HIPCC_FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-shared", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 code generation
               "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]   # the direct-load asm declares that it writes m0


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile with hipcc (cross-compiles without a GPU).  force=False skips an up-to-date library."""
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in DEPS):
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + HIPCC_FLAGS + ["-o", LIB, SRC]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(ln for ln in res.stderr.splitlines() if noise not in ln)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
