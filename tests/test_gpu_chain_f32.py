"""Narrow fp32 models, whole passes and whole draft chains in one launch (csrc/chain_f32.h), against the oracle: rows of less than a lane's piece
per lane up to two, fewer and more heads than wavefronts, head_dim 32 and 64, grouped queries, both activations, FFN widths beside and
past the prefetched columns, vocabularies that the draw takes in two chunks, in eight and not at all, the most layers and one more,
blocks of 2 .. 16 rows, contexts across the chunks of 32 and 64 positions and past the limit, drafters with a backlog of their own."""
import pytest

import oracle
import paper_2604_05417_amd as M
import workloads as W
from lockstep import LockStep

pytestmark = pytest.mark.gpu
TOL = 1e-4

#        d, heads, kv heads, d_ffn, act, vocab, layers, prompt, gamma, T, shared cache
SHAPES = [(32, 1, 1, 4, W.GELU, 8, 1, 3, 1, 1.0, True), (96, 3, 1, 100, W.SWIGLU, 260, 2, 29, 3, 0.7, False), (128, 4, 4, 512, W.GELU, 512, 2, 16, 4, 1.0, True),
          (128, 2, 1, 516, W.SWIGLU, 516, 8, 61, 7, 0.0, True), (160, 5, 5, 1028, W.GELU, 2048, 9, 33, 8, 1.0, False), (288, 9, 3, 260, W.SWIGLU, 2052, 2, 7, 5, 1.0, True),
          (256, 8, 2, 2048, W.SWIGLU, 1000, 2, 490, 15, 1.0, True), (512, 8, 8, 2048, W.GELU, 300, 2, 62, 15, 0.0, False), (512, 16, 4, 2044, W.SWIGLU, 1500, 3, 120, 2, 0.7, True)]


def build(i, alone=False):
    d, H, KH, f, act, V, L, n, gamma, T, shared = SHAPES[i]
    td = W.model_desc(L, d, H, KH, f, V, act, W.FP32)
    tw = W.gen_weights(td, 0)
    if shared:
        drafters = [(dict(td, n_layers=max(1, L - 1 - k)), tw[: 1 + 9 * max(1, L - 1 - k)] + tw[-2:]) for k in range(2)]
    else:
        dd = W.model_desc(1, 96, 3, 1, 40, V, W.SWIGLU, W.FP32)
        drafters = [(dd, W.gen_weights(dd, 7 + k)) for k in range(2)]
    max_ctx, prompt = n + 120, W.prompt_tokens(n, V, 3)
    g = M.MetaSD((td, tw), drafters, gamma_max=gamma, max_ctx=max_ctx, temperature=T, seed=4, share_target_kv=shared)
    if alone:
        return g, prompt, gamma, None
    ot = oracle.Model(td, W.to_numpy(tw), max_ctx)
    od = [oracle.Model(dd, W.to_numpy(w), max_ctx, share_kv_with=ot if shared else None) for dd, w in drafters]
    g.set_context(prompt)
    return g, prompt, gamma, LockStep(g, ot, od, prompt, gamma, T, 4, 1.0, logit_tol=TOL)


@pytest.mark.parametrize("separate", [False, True])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_chain_f32(i, separate):
    g, _, _, ls = build(i)
    if separate:                                   # launches that are timed one by one are the separate ones
        g.profile(1)
    for arm in (0, 1, 1, 0):
        ls.round(arm)
    g.close()
    assert ls.stats["max_dp"] <= TOL and ls.stats["max_dq"] <= TOL and ls.stats["ties_shared"] <= 1, ls.stats


def test_chain_f32_bounded_wait(monkeypatch):
    """With the bound of the waits forced to zero every workgroup gives up at once: the round reports an error, nothing hangs or reads out of
    bounds, and a new context works again."""
    g, prompt, gamma, _ = build(2, alone=True)
    g.set_context(prompt, kv_prefilled=True)
    monkeypatch.setenv("METASD_GEMM_SPIN_LIMIT", "0")
    g.draft(0, gamma)
    g.verify(gamma)
    with pytest.raises(M.MetaSDError) as e:
        g.accept(gamma)
    assert e.value.code == -4
    monkeypatch.delenv("METASD_GEMM_SPIN_LIMIT")
    g.close()
    g, _, _, ls = build(2)
    ls.round(0)
    g.close()
