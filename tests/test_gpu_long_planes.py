"""Contexts so long that one head's K or V plane is more than 4 GiB (2^24 positions of 128 bf16 values): what the attention kernels read at the
far end of it.

All keys of the prefix are zero, so every position has the same weight, and it does not matter where in the prefix the few values that are
not zero stand: with them in front and with them behind position 2^24 the logits have to agree.  An offset that wraps at 4 GiB reads the
front of the plane instead."""
import numpy as np
import pytest

import paper_2604_05417_amd as M
import workloads as W

pytestmark = pytest.mark.gpu
FAR = 1 << 24
N_SPIKE = 96
PROMPT = W.prompt_tokens(FAR + 200, 256, 3)
# The prefix is summed exactly on both sides (weights of one, values that are powers of two, partial sums below 2^24); what differs is where
# the block's own positions, of weight near one, meet the rest: a few fp32 roundings, and behind them the bf16 terms of the activations
# (2^-16 of values of size 1).
TOL = 2e-4


def fill(g, at, seq=None):
    """Keys zero, values zero but for N_SPIKE positions from `at` on: their mean over the prefix is 0.375."""
    for kv in {t.data_ptr(): t for t in [g.kv_target] + g.kv_drafters}.values():
        kv.zero_()
        (kv if seq is None else kv[seq])[:, 1, :, at: at + N_SPIKE] = 65536.0


def check(run):
    near, far, none = run(5), run(FAR + 40), run(None)
    for a, b, z in zip(near, far, none):
        assert np.abs(a - b).max() <= TOL, np.abs(a - b).max()
        assert np.abs(a - z).max() >= 100 * TOL                   # the values do reach the logits


def model(layers):
    td = W.model_desc(layers, 128, 1, 1, 160, 256, W.SWIGLU, W.BF16)
    return td, W.gen_weights(td, 0)


@pytest.mark.parametrize("batch", [1, 2])
def test_short_blocks_behind_4_gib(batch):
    td, tw = model(1)
    g = M.MetaSD((td, tw), [(td, tw)], gamma_max=5, max_ctx=FAR + 256, temperature=0.0, seed=1, batch=batch, share_target_kv=True)

    def run(at):
        if at is None:
            g.kv_target.zero_()
        else:
            fill(g, at, 0 if batch > 1 else None)
        g.set_context(PROMPT, kv_prefilled=True)
        if batch > 1:
            g.set_context(PROMPT[:50], kv_prefilled=True, seq=1)
        g.draft(0, 5)
        g.verify(5)
        out = [g.peek(k, 5)[0].cpu().numpy() if batch > 1 else g.peek(k).cpu().numpy() for k in ("P", "Q")]
        g.accept(5)
        return out
    check(run)
    g.close()


def test_long_block_behind_4_gib(monkeypatch):
    """A drafter that sat out eight rounds of 16 tokens reads them as one long block."""
    monkeypatch.setenv("METASD_ATT_CPW", "64")                    # the rounds before it over the whole chip
    td, tw = model(2)
    g = M.MetaSD((td, tw), [(td, tw), (td, W.gen_weights(td, 9))], gamma_max=15, max_ctx=FAR + 512, temperature=0.0, seed=1, share_target_kv=True)

    def run(at):
        if at is None:
            for kv in (g.kv_target, g.kv_drafters[1]):
                kv.zero_()
        else:
            fill(g, at)
        g.set_context(PROMPT, kv_prefilled=True)
        for _ in range(8):
            g.draft(0, 15)
            g.verify(15)
            assert g.accept(15)[0] == 15                          # the drafter is the target
        g.draft(1, 1)
        q = g.peek("Q")[:1].cpu().numpy()
        g.verify(1)
        g.accept(1)
        return [q]
    check(run)
    g.close()
