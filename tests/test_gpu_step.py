"""The GEMM of short blocks with its K reduction inside the workgroup (csrc/step.h) at the sizes where its split changes: block heights
1 .. 16, K ranges that leave wavefronts without a slice or with a short one, odd numbers of 32-wide chunks (no half tiles), tile counts
above and below the number of CUs, more tiles than one pass of a workgroup takes, GELU, grouped queries; and the same blocks through
the kernels that take over when it is switched off.  Against the oracle, round by round."""
import pytest

import workloads as W
from test_gpu_bf16 import TOL, run_lockstep

pytestmark = pytest.mark.gpu

# target (d_model, heads, kv heads, d_ffn, act, vocab), drafter (d_model, heads, d_ffn, act), gamma
SHAPES = [
    ((512, 8, 8, 544, W.SWIGLU, 528), (128, 2, 160, W.GELU), 7),          # 16 chunks: one per wavefront; 17 chunks of d_ffn
    ((544 + 32, 9, 3, 3104, W.GELU, 4112), (192, 3, 96, W.SWIGLU), 4),    # 18 chunks over 16 wavefronts; 97 chunks
    ((2048, 32, 8, 1024, W.SWIGLU, 1040), (2048, 16, 8192, W.SWIGLU), 2),  # widest rows and d_ffn the short path takes
    ((512, 4, 4, 33024, W.SWIGLU, 512), (256, 4, 288, W.SWIGLU), 5),      # more pairs of tiles than one pass of 256 workgroups
    ((3072, 24, 24, 4096, W.SWIGLU, 1024), (128, 2, 160, W.SWIGLU), 7),   # 8 rows of 3072: four float4 columns and more per lane
    ((4096, 32, 8, 1024, W.SWIGLU, 512), (128, 2, 160, W.SWIGLU), 7),     # 8 rows of 4096: all eight columns, the most LDS it takes
    ((512, 8, 8, 544, W.SWIGLU, 528), (512, 8, 544, W.GELU), 11),         # 9 - 16 rows: one chunk per wavefront, 17 chunks of d_ffn
    ((2048, 32, 8, 1024, W.SWIGLU, 1040), (576, 9, 3104, W.GELU), 15),    # .. the most LDS it takes; half tiles and odd numbers of chunks
    ((2048, 16, 16, 4128, W.GELU, 1040), (1024, 8, 8192, W.SWIGLU), 8),   # .. d_ffn one chunk longer than the step GEMM adds; gate | up above 256 units
    ((2080, 65, 13, 544, W.SWIGLU, 512), (128, 2, 160, W.SWIGLU), 8),     # .. rows too wide by one chunk: the split-K path
    ((4224, 33, 11, 1024, W.SWIGLU, 512), (128, 2, 160, W.SWIGLU), 7),    # 8 rows of 4224 do not fit: verified on the split-K path
]


@pytest.mark.parametrize("fuse", ["1", "0"])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_step_gemm_shapes(i, fuse, monkeypatch):
    monkeypatch.setenv("METASD_FUSE_SMALL", fuse)
    (d, H, KH, f, act, V), (dd, dH, df, dact), gamma = SHAPES[i]
    td = W.model_desc(1, d, H, KH, f, V, act, W.BF16)
    drafters = []
    for k in range(2):
        desc = W.model_desc(1, dd, dH, dH, df, V, dact, W.BF16)
        drafters.append((desc, W.gen_weights(desc, 100 + k)))
    cfg = dict(target=(td, W.gen_weights(td, 0)), drafters=drafters, gamma=gamma, prompt=W.prompt_tokens(19, V, 3), beta=1.0, seed=5, max_ctx=19 + 80)
    # arms forced: a drafter that returns has a backlog of up to 2 (gamma + 1) rows in front of its first step
    st = run_lockstep(cfg, 1.0, rounds=4, kv_prefilled=False, force_arms=[0, 1, 1, 0])
    assert st["max_dp"] <= TOL and st["max_dq"] <= TOL and st["ties_shared"] <= 1, st
