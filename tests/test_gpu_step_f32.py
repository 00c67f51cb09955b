"""fp32 models on the five-launch layer (csrc/step_f32.h) and on the ten-launch layer it replaces for narrow rows, at the sizes where the
former changes: rows shorter than a wavefront's float4 column, of one and a half columns, of exactly two and just over (ten launches);
output counts that are no multiple of four wavefronts; block heights in every unrolling; head_dim 32 and 64, grouped queries, SwiGLU and
GELU; contexts of one attention chunk (no merge), across the boundary of 128 positions, and of three.  Against the oracle."""
import pytest

import oracle
import paper_2604_05417_amd as M
import workloads as W
from lockstep import LockStep

pytestmark = pytest.mark.gpu
TOL = 1e-4

#        d, heads, kv heads, d_ffn, act, vocab, prompt, gamma
SHAPES = [(64, 2, 1, 36, W.SWIGLU, 36, 5, 1), (192, 6, 2, 100, W.GELU, 264, 122, 3), (384, 6, 6, 516, W.SWIGLU, 1000, 7, 4),
          (512, 8, 4, 1540, W.GELU, 512, 300, 7), (512, 16, 16, 260, W.SWIGLU, 2052, 16, 15), (576, 9, 3, 264, W.SWIGLU, 516, 30, 5)]


@pytest.mark.parametrize("fuse", ["1", "0"])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_f32_layers(i, fuse, monkeypatch):
    monkeypatch.setenv("METASD_FUSE_SMALL", fuse)
    d, H, KH, f, act, V, n, gamma = SHAPES[i]
    td = W.model_desc(2, d, H, KH, f, V, act, W.FP32)
    dd = W.model_desc(1, 96, 3, 1, 40, V, W.SWIGLU, W.FP32)
    tw, dw = W.gen_weights(td, 0), [W.gen_weights(dd, 7 + k) for k in range(2)]
    max_ctx, prompt = n + 120, W.prompt_tokens(n, V, 3)
    g = M.MetaSD((td, tw), [(dd, w) for w in dw], gamma_max=gamma, max_ctx=max_ctx, temperature=1.0, seed=4)
    ot = oracle.Model(td, W.to_numpy(tw), max_ctx)
    od = [oracle.Model(dd, W.to_numpy(w), max_ctx) for w in dw]
    g.set_context(prompt)
    ls = LockStep(g, ot, od, prompt, gamma, 1.0, 4, 1.0, logit_tol=TOL)
    for arm in (0, 1, 1, 0):
        ls.round(arm)
    g.close()
    assert ls.stats["max_dp"] <= TOL and ls.stats["max_dq"] <= TOL and ls.stats["ties_shared"] <= 1, ls.stats


@pytest.mark.parametrize("d,H,KH,n,gamma", [(96, 3, 1, 30, 1), (256, 8, 8, 55, 7), (512, 16, 4, 117, 5), (256, 4, 2, 46, 15), (128, 2, 2, 60, 3)])
def test_f32_attention_with_output_projection(d, H, KH, n, gamma):
    """Attention and output projection in one launch (contexts of up to 128 positions at head_dim 32, 64 at head_dim 64), with rounds that
    grow past 64 and 128 positions: the two forms of the kernel and the path behind them, every block height, grouped queries."""
    td, dd = W.model_desc(2, d, H, KH, 132, 260, W.GELU, W.FP32), W.model_desc(1, d, H, KH, 68, 260, W.SWIGLU, W.FP32)
    tw, dw = W.gen_weights(td, 0), W.gen_weights(dd, 7)
    max_ctx, prompt = n + 5 * (gamma + 1) + 8, W.prompt_tokens(n, 260, 3)
    g = M.MetaSD((td, tw), [(dd, dw)], gamma_max=gamma, max_ctx=max_ctx, temperature=1.0, seed=4)
    ot, od = oracle.Model(td, W.to_numpy(tw), max_ctx), [oracle.Model(dd, W.to_numpy(dw), max_ctx)]
    g.set_context(prompt)
    ls = LockStep(g, ot, od, prompt, gamma, 1.0, 4, 1.0, logit_tol=TOL)
    for _ in range(4):
        ls.round(0)
    g.close()
    assert ls.stats["max_dp"] <= TOL and ls.stats["max_dq"] <= TOL and ls.stats["ties_shared"] <= 1, ls.stats
