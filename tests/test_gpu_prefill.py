"""Prefill of long prompts in large row blocks: every K/V entry the target's cache holds afterwards against a plain PyTorch
fp32 forward of the same model, at the edges of the row tiles and of the blocks, and the rounds that follow against the oracle."""
import math

import pytest
import torch

import paper_2604_05417_amd as M
import workloads as W
from test_gpu_batch import batch_pair, make_lockstep
from lockstep import LockStep
from test_gpu_bf16 import oracle_models, run_lockstep

pytestmark = pytest.mark.gpu
TOL = 3e-2


def kv_reference(desc, w, tokens, h0=None):
    """K and V of every position and layer, [layer, 2, kv_head, n, hd] fp32 (rounded to bf16 where the cache rounds), and the residual
    rows behind the last layer.  h0: residual rows in front of the first, the embedding if None."""
    d, H, KH, L = desc["d_model"], desc["n_heads"], desc["n_kv_heads"], desc["n_layers"]
    hd, n, dev = d // H, len(tokens), w[0].device
    f = [None if t is None else t.float() for t in w]
    norm = lambda x, g: x * torch.rsqrt(x.square().mean(-1, keepdim=True) + desc["rms_eps"]) * g
    ang = (torch.arange(n, device=dev, dtype=torch.float64)[:, None] *
           desc["rope_theta"] ** (-2.0 * torch.arange(hd // 2, device=dev, dtype=torch.float64) / hd))
    cs, sn = ang.cos().float()[None], ang.sin().float()[None]

    def rot(x):
        a, b = x[..., : hd // 2], x[..., hd // 2:]
        return torch.cat([a * cs - b * sn, a * sn + b * cs], -1)

    h = f[0][torch.as_tensor(tokens, device=dev, dtype=torch.int64)] if h0 is None else h0
    mask = torch.ones((n, n), dtype=torch.bool, device=dev).tril()
    out = []
    for i in range(L):
        g1, wq, wk, wv, wo, g2, wg, wu, wd = f[1 + 9 * i: 10 + 9 * i]
        x = norm(h, g1)
        heads = lambda y, nh: y.view(n, nh, hd).transpose(0, 1)
        q = rot(heads(x @ wq.T, H))
        k = rot(heads(x @ wk.T, KH)).bfloat16().float()
        v = heads(x @ wv.T, KH).bfloat16().float()
        out.append(torch.stack([k, v]))
        kk, vv = (t.repeat_interleave(H // KH, 0).contiguous() for t in (k, v))
        s = torch.matmul(q, kk.transpose(1, 2).contiguous()) / math.sqrt(hd)
        o = torch.matmul(torch.softmax(s.masked_fill(~mask, -math.inf), -1), vv)
        h = h + o.transpose(0, 1).reshape(n, H * hd) @ wo.T
        x = norm(h, g2)
        h = h + (torch.nn.functional.silu(x @ wg.T) * (x @ wu.T)) @ wd.T
    return torch.stack(out), h


def assert_kv(kv, ref):
    # both sides round to bf16 (half an ulp each, 2^-8 of the value) what they hold to about 1e-3 of the rows' rms
    bad = (kv - ref).abs() > ref.abs() * 2.0 ** -7 + 2e-3 * ref.square().mean().sqrt()
    assert not bad.any(), (bad.nonzero()[:4].tolist(), int(bad.sum()))


def check_prefill(desc, n, batch=1, seed=5):
    tw = W.gen_weights(desc, seed, device="cuda")
    drafters = [W.early_exit_drafter(desc, tw, 1, 0.01, 9)]
    g = M.MetaSD((desc, tw), drafters, gamma_max=3, max_ctx=n + 8, temperature=1.0, seed=1, batch=batch, share_target_kv=True)
    for b in range(batch):
        tok = W.prompt_tokens(n - b, desc["vocab"], 3 + b)
        g.set_context(tok, seq=b)
        torch.cuda.synchronize()
        kv = (g.kv_target[b] if batch > 1 else g.kv_target).float()
        ref, _ = kv_reference(desc, tw, tok[:-1])
        m = n - b - 1
        assert_kv(kv[:, :, :, :m], ref)
        assert (kv[:, :, :, m:] == 0).all()                       # nothing past the prompt
    g.close()


HD64 = W.model_desc(3, 512, 8, 2, 736, 528, W.SWIGLU, W.BF16)
HD128 = W.model_desc(2, 512, 4, 4, 1056, 528, W.SWIGLU, W.BF16)


@pytest.mark.parametrize("n", [18, 33, 65, 66, 128, 129, 130, 257, 258, 600])
@pytest.mark.parametrize("desc", [HD64, HD128], ids=["hd64_gqa", "hd128"])
def test_prefill_leaves_the_models_kv(desc, n):
    check_prefill(desc, n)


TILES = [(4, 12), (3, 16), (3, 12), (3, 8), (2, 16), (2, 12), (2, 8), (2, 6), (1, 16), (1, 12), (1, 8), (1, 4)]


@pytest.mark.parametrize("rb,tpb", TILES)
def test_every_tile_of_the_many_row_gemm(rb, tpb, monkeypatch):
    """Each workgroup tile (64 rb rows x tpb feature tiles), forced: one row less than a row block, a full one, one row more, and
    a second block with a ragged end; 48 / 92 / 32 tiles and 16 / 23 chunks of K, with and without a K split."""
    monkeypatch.setenv("METASD_ROWS_RB", str(rb))
    monkeypatch.setenv("METASD_ROWS_TPB", str(tpb))
    for rows in (64 * rb - 1, 64 * rb, 64 * rb + 1, 128 * rb + 17):
        check_prefill(HD64, rows + 1)


def test_prefill_of_more_than_one_block():
    check_prefill(HD64, 2048 + 21)                                # a block of 2048 rows and one of 20


@pytest.mark.parametrize("last", [1, 16, 17])
@pytest.mark.parametrize("desc", [HD64, HD128], ids=["hd64_gqa", "hd128"])
def test_prefill_whose_last_block_is_short(desc, last):
    """A block of 2048 rows and one of few: up to 16 rows take the GEMM of short blocks, with activations as two arrays."""
    check_prefill(desc, 2048 + last + 1)


def test_features_and_a_drafter_head_over_a_block_and_a_short_one():
    """A prompt of 2048 + 9 + 1 tokens: the target's features of every position, and the K/V of a head that reads the prompt with them."""
    n = 2048 + 9 + 1
    tw = W.gen_weights(HD64, 5, device="cuda")
    dd, dw, fc = W.feature_head_drafter(HD64, tw, 0, 0.02, 300)
    g = M.MetaSD((HD64, tw), [(dd, dw)], gamma_max=3, max_ctx=n + 8, temperature=1.0, seed=1, heads={0: fc})
    tok = W.prompt_tokens(n, HD64["vocab"], 3)
    g.set_context(tok)
    g.draft(0, 1)
    torch.cuda.synchronize()
    _, feat = kv_reference(HD64, tw, tok[:-1])
    got = g.peek("feat")[: n - 1]
    # fp32 on both sides; a K/V entry that rounded to the other neighbour moves them by less than the 2e-3 of assert_kv
    assert ((got - feat).abs() <= 2e-3 * feat.square().mean().sqrt() + 2.0 ** -9 * feat.abs()).all()
    emb = tw[0].float()[torch.as_tensor(tok[:-1], device="cuda", dtype=torch.int64)]
    before = torch.cat([torch.zeros_like(feat[:1]), got[:-1]])    # the features the head was given
    ref, _ = kv_reference(dd, dw, tok[:-1], torch.cat([emb, before], 1) @ fc.float().cuda().T)
    assert_kv(g.kv_drafters[0].float()[:, :, :, : n - 1], ref)
    g.close()


@pytest.mark.parametrize("desc", [W.model_desc(2, 1024, 16, 4, 352, 528, W.SWIGLU, W.BF16), W.model_desc(2, 2048, 16, 16, 352, 528, W.SWIGLU, W.BF16)],
                         ids=["hd64", "hd128"])
def test_prefill_with_32_rows_per_wavefront(desc):
    check_prefill(desc, 2048 + 1)                                 # 16 row blocks of 128 x 16 heads fill the chip


def test_prefill_of_a_sequence_in_a_batch():
    check_prefill(HD64, 140, batch=3)


@pytest.mark.parametrize("n", [37, 300])
def test_rounds_after_a_long_prefill_and_drafter_catch_up(n):
    cfg = W.config4(n_layers=2, ctx=n, n_new=64, K=2, d_model=256, n_heads=4, d_ffn=512, vocab=1024, dd_model=128, dn_heads=2, dd_ffn=160)
    cfg["gamma"], cfg["max_ctx"] = 4, n + 60
    st = run_lockstep(cfg, 1.0, rounds=4, kv_prefilled=False)
    assert st["max_dp"] <= TOL and st["max_dq"] <= TOL and st["ties_shared"] <= 1, st


@pytest.mark.parametrize("ctx,idle,big", [(600, 2, True), (3000, 2, False), (3000, 3, True)])
def test_short_backlog_at_a_long_context(ctx, idle, big):
    """A drafter that was idle for `idle` rounds of nine tokens returns: its 18 or 27 unseen rows go through in one block, or, where the
    context is long against them, in blocks of 16 (one block walks 3000 positions with two workgroups).  Drafters are copies of the
    target with the same K/V, so that every draft token is accepted."""
    desc = W.model_desc(2, 256, 2, 2, 512, 528, W.SWIGLU, W.BF16)
    w = W.gen_weights(desc, 0)
    cfg = dict(target=(desc, w), drafters=[(desc, w), (desc, w)], max_ctx=ctx + 64)
    g = M.MetaSD((desc, w), cfg["drafters"], gamma_max=8, max_ctx=cfg["max_ctx"], temperature=0.0, seed=1)
    ot, od = oracle_models(cfg)
    kv = W.kv_fill(desc, ctx - 1, 7, device="cuda")
    for i, t in enumerate(kv):
        for gpu, om in zip([g.kv_target] + g.kv_drafters, [ot] + od):
            gpu[:, i, :, : ctx - 1] = t
            om.kv(i)[:, :, : ctx - 1] = t.float().cpu().numpy()
    prompt = W.prompt_tokens(ctx, desc["vocab"], 3)
    g.set_context(prompt, kv_prefilled=True)
    ls = LockStep(g, ot, od, prompt, 8, 0.0, 1, 1.0, logit_tol=TOL, kv_prefilled=True)
    for _ in range(idle):
        ls.round(0)
    assert ls.l == ctx + 9 * idle
    g.profile(512)
    ls.round(1)
    rows = max(x["m"] for x in g.profile_shapes(target_only=False))      # of the GEMM launches of this round
    assert rows == (9 * idle if big else 16), rows
    g.close()


def test_ragged_batch_with_long_drafter_backlogs():
    cfg = W.config4(n_layers=2, ctx=40, n_new=64, K=2, d_model=256, n_heads=4, d_ffn=512, vocab=1024, dd_model=128, dn_heads=2, dd_ffn=160)
    cfg["gamma"], cfg["max_ctx"] = 3, 420
    prompts = [W.prompt_tokens(n, 1024, 70 + i) for i, n in enumerate((350, 12, 120))]
    g, seqs = batch_pair(cfg, 1.0, prompts, TOL)
    bl = make_lockstep(g, cfg, seqs, prompts, 1.0, TOL)
    for _ in range(4):
        bl.round()
    g.close()
    for ls in bl.seqs:
        assert ls.stats["max_dp"] <= TOL and ls.stats["max_dq"] <= TOL and ls.stats["ties_shared"] <= 1, ls.stats
