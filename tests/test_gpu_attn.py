"""Attention of short blocks at the sizes where its split can go wrong: contexts around a sub-block (32 positions) and a pass of a
workgroup (128), every branch of the rule that splits them (csrc/attn_plan.h; counts below for 256 CUs), one to four query heads of a K/V
head packed into one operand, 1 to 16 rows."""
import pytest

import workloads as W
from test_gpu_bf16 import run_lockstep

pytestmark = pytest.mark.gpu
# An element of the K/V cache that rounds to the other bf16 neighbour on one side is off by 2^-8 of itself; the logits of these
# two-layer models move by less than that, everything else (two bf16 terms per activation: 2^-16) is far below.
TOL = 4e-3


@pytest.mark.parametrize("d,heads,kv,gamma,ctx,passes", [
    # heads of 64; query heads of a K/V head packed for the drafter's row and for the verified rows
    (512, 8, 2, 1, 30, 0), (512, 8, 2, 3, 31, 0), (512, 8, 2, 7, 121, 0),         # 4 and 4, 4 and 4, 4 and 2; one record
    (512, 8, 2, 7, 127, 1), (512, 8, 2, 3, 513, 1), (512, 8, 2, 15, 129, 1),      # 4 and 2, 4 and 4, 4 and 1; two, five and two records, forced
    (768, 6, 2, 4, 200, 1), (768, 6, 2, 1, 300, 0),                               # heads of 128, 3 packed; two and three records
    # one query head per K/V head
    (512, 8, 8, 5, 640, 0), (512, 8, 8, 5, 641, 2), (512, 8, 8, 11, 1100, 0),     # five (drafter) and six, three (forced), five of two passes
    (512, 8, 8, 5, 8100, 0),                                                      # few heads and a long context: 16 records
    (2048, 32, 32, 5, 850, 0),                                                    # 32 heads: four records of two passes instead of seven of one
    (512, 4, 4, 5, 33, 0), (512, 4, 4, 5, 257, 0), (512, 4, 4, 12, 400, 1),       # heads of 128: one, three and four records
])
def test_attention_splits(d, heads, kv, gamma, ctx, passes, monkeypatch):
    if passes:
        monkeypatch.setenv("METASD_ATT_CPW", str(passes))
    td = W.model_desc(2, d, heads, kv, 512, 1024, W.SWIGLU, W.BF16)
    tw = W.gen_weights(td, 0)
    cfg = dict(target=(td, tw), drafters=[W.early_exit_drafter(td, tw, 1, 0.01, 100)], gamma=gamma, prompt=W.prompt_tokens(ctx, 1024, 3),
               beta=1.0, seed=1, kv_seed=7, max_ctx=ctx + 2 * gamma + 40)
    st = run_lockstep(cfg, 1.0, rounds=2, kv_prefilled=True)
    assert st["max_dp"] <= TOL and st["max_dq"] <= TOL and st["ties_shared"] <= 1, st
