"""Workloads on which the speed of this library is followed, through its public entry points.

Four kinds of work, each as a user's program calls it:
  query   one query on a batch-1 context: metasd_set_context (the prompt prefilled by the library, or its KV cache already
          there), then rounds of bandit_select / draft / verify / accept / bandit_update (or tree rounds)
  batch   the same for several sequences that share a context and advance in lock-step
  accept  the stand-alone accept step on rows of logits the caller holds
Model shapes are the repository's own: "7b" with five two-layer drafters, "1b" (grouped queries) with four early-exit
drafters, "tiny" in fp32.

Weights.  Untrained weights give next-token laws that are flat over the vocabulary; what a trained pair of models has is a law
with most of its mass on one token, on which target and drafter agree more often than not.  The models here get that from
their embedding and head: every token has one likely successor (a permutation of the vocabulary), and drafter k agrees with
the target on a share of the tokens.  It also keeps the tokens of a query from hanging on the last bits of a logit.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2604_05417_amd as M

DEV = "cuda:0"
SWIGLU, GELU, BF16, FP32 = 1, 0, 1, 0
SUCC = 45.0             # d_model times the weight with which a token's embedding enters the head row of its successor
AGREE = (0.9, 0.8, 0.7, 0.6, 0.5)


def _desc(layers, d, heads, kv_heads, ffn, vocab, act=SWIGLU, dtype=BF16):
    return dict(n_layers=layers, d_model=d, n_heads=heads, n_kv_heads=kv_heads, d_ffn=ffn, vocab=vocab, act=act, dtype=dtype,
                rms_eps=1e-5, rope_theta=10000.0)


TARGET = {"tiny": _desc(2, 128, 4, 4, 512, 512, GELU, FP32), "1b": _desc(16, 2048, 32, 8, 8192, 32000),
          "7b": _desc(32, 4096, 32, 32, 11008, 32000)}
EARLY_EXIT = {"tiny": (1, 1, 1), "1b": (2, 4, 6, 8)}        # layers of the target that drafter k runs
DRAFTER = {"7b": _desc(2, 768, 12, 12, 3072, 32000)}        # five drafters with weights of their own

# a draft tree of 13 nodes and depth 5: three candidates after the root, two after the likeliest nodes of the next levels
TREE = dict(parent=[-1, 0, 0, 0, 1, 1, 2, 4, 4, 5, 7, 7, 10], rank=[0, 0, 1, 2, 0, 1, 0, 0, 1, 0, 0, 1, 0], depth=5)


def listed():
    def query(name, shape, ctx, gamma, rounds, prefilled, T=1.0, tree=False):
        return dict(name=name, kind="query", shape=shape, ctx=ctx, gamma=gamma, rounds=rounds, prefilled=prefilled, T=T, tree=tree)

    def batch(name, shape, batch, ctx, gamma, rounds, prefilled, T):
        return dict(name=name, kind="batch", shape=shape, batch=batch, ctx=ctx, gamma=gamma, rounds=rounds, prefilled=prefilled, T=T)

    def accept(name, rows, gamma, vocab, T):
        return dict(name=name, kind="accept", rows=rows, gamma=gamma, vocab=vocab, T=T)

    return [
        query("query_tiny_fp32", "tiny", 16, 4, 12, False),           # the smallest model: a whole short query, all launches
        query("start_1b", "1b", 512, 5, 1, False),                    # a new query: prefill of its prompt and the first round
        query("start_7b", "7b", 1500, 5, 1, False),                   # .. with separate drafters, whose first round reads the prompt too
        query("decode_1b", "1b", 777, 5, 8, True),                    # generation in steady state, early-exit drafters
        query("decode_7b", "7b", 2048, 5, 8, True),                   # the headline: one sequence at context 2048
        query("decode_7b_long", "7b", 8000, 11, 6, True),             # long context, long chains, backlogs of more than 8 rows
        query("tree_7b", "7b", 2048, 13, 6, True, tree=True),         # multi-candidate rounds
        batch("batch_7b", "7b", 32, 2048, 7, 5, True, 0.7),           # serving: 32 sequences, 256 verification rows
        batch("batch_1b", "1b", 5, 333, 3, 5, False, 1.0),            # a small ragged batch, prompts prefilled by the library
        accept("accept_1", 1, 5, 32000, 1.0),                         # the accept step of one sequence
        accept("accept_64", 64, 5, 32000, 1.0),                       # .. of 64
        accept("accept_250", 250, 7, 32000, 0.7),                     # .. of many, temperature other than 1
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("query", "query", "query", "batch", "accept", "accept"))
    if kind == "accept":
        gamma = rng.randint(1, 15)
        return dict(kind=kind, rows=_log_int(rng, 1, 2000 // (gamma + 1)), gamma=gamma, vocab=4 * _log_int(rng, 128, 8192),
                    T=rng.choice((0.0, 0.7, 1.0)))
    if kind == "batch":
        shape, gamma = rng.choice(("1b", "7b")), rng.randint(1, 7)
        prefilled = rng.random() < 0.6
        return dict(kind=kind, shape=shape, batch=rng.randint(2, 32 if prefilled else 4), ctx=_log_int(rng, 64, 2000 if prefilled else 320),
                    gamma=gamma, rounds=rng.randint(1, 5), prefilled=prefilled, T=rng.choice((0.0, 0.7, 1.0)))
    shape, prefilled, tree = rng.choice(("tiny", "1b", "7b", "7b")), rng.random() < 0.5, rng.random() < 0.2
    hi = 120 if shape == "tiny" else (8000 if prefilled else 1400)
    return dict(kind=kind, shape=shape, ctx=_log_int(rng, 8, hi), gamma=13 if tree else rng.randint(1, 15), rounds=rng.randint(1, 6),
                prefilled=prefilled, T=rng.choice((0.0, 1.0)), tree=tree)


# ------------------------------------------------------------------------------------------- models

def _weights(desc, gen):
    """Random tables of a model; the projections into the residual stream are scaled down with the depth, the embedding has unit
    variance, so that the residual stream still carries the token at the last layer."""
    d, H, KH, f, V, L = (desc[k] for k in ("d_model", "n_heads", "n_kv_heads", "d_ffn", "vocab", "n_layers"))
    hd, dt = d // H, torch.bfloat16 if desc["dtype"] == BF16 else torch.float32

    def rnd(*shape, std=0.02, mean=0.0):
        return torch.empty(shape, dtype=dt, device=DEV).normal_(mean, std, generator=gen)

    res = 0.02 / math.sqrt(2 * L)
    w = [rnd(V, d, std=1.0)]
    for _ in range(L):
        w += [rnd(d, mean=1.0), rnd(H * hd, d), rnd(KH * hd, d), rnd(KH * hd, d), rnd(d, H * hd, std=res), rnd(d, mean=1.0),
              rnd(f, d) if desc["act"] == SWIGLU else None, rnd(f, d), rnd(d, f, std=res)]
    return w + [rnd(d, mean=1.0), None]


def _head(embed, succ, gen):
    d = embed.shape[1]
    head = torch.empty(embed.shape, dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=gen)
    head[succ] += (SUCC / d) * embed.float()
    return head.to(embed.dtype)


def _disagree(succ, share, gen):
    """succ with the successors of (1 - share) of the tokens exchanged among them."""
    V = succ.numel()
    at = torch.randperm(V, generator=gen, device=DEV)[int(share * V):]
    out = succ.clone()
    out[at] = succ[at.roll(1)]
    return out


def _models(shape, gen):
    td = TARGET[shape]
    tw = _weights(td, gen)
    succ = torch.randperm(td["vocab"], generator=gen, device=DEV)
    tw[-1] = _head(tw[0], succ, gen)
    drafters = []
    for k in range(len(EARLY_EXIT.get(shape, AGREE))):
        mine = _disagree(succ, AGREE[k], gen)
        if shape in EARLY_EXIT:
            n = EARLY_EXIT[shape][k]
            drafters.append((dict(td, n_layers=n), tw[: 1 + 9 * n] + [tw[-2], _head(tw[0], mine, gen)]))
        else:
            dw = _weights(DRAFTER[shape], gen)
            dw[-1] = _head(dw[0], mine, gen)
            drafters.append((DRAFTER[shape], dw))
    return (td, tw), drafters


# ------------------------------------------------------------------------------------------- cases

def _lengths(case):
    """Prompt lengths of the sequences of a case: a batch is ragged."""
    n = case.get("batch", 1)
    return [case["ctx"] - (3 * b) % max(1, case["ctx"] // 4) for b in range(n)]


def _max_ctx(case):
    return case["ctx"] + (case["gamma"] + 1) * case["rounds"] + 32


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    if case["kind"] == "accept":
        rows, gamma, V = case["rows"], case["gamma"], case["vocab"]
        P = torch.empty((rows, gamma + 1, V), device=DEV).normal_(0.0, 2.0, generator=gen)
        Q = P[:, :gamma] + torch.empty((rows, gamma, V), device=DEV).normal_(0.0, 1.0, generator=gen)
        # draft tokens are draws from the drafter's law (the largest of logit + Gumbel noise), the likeliest when greedy
        noise = torch.empty_like(Q).exponential_(generator=gen).clamp_min_(1e-20).log_().neg_() * case["T"]
        d = (Q + noise).argmax(-1).to(torch.int32).contiguous()
        res = torch.zeros((3, rows), dtype=torch.int32, device=DEV)
        out = dict(n_acc=res[0], token=res[1], mask=res[2], bd=torch.zeros((rows, gamma), dtype=torch.float64, device=DEV),
                   scratch=torch.zeros(rows * (gamma + 1) * 336, dtype=torch.uint8, device=DEV))
        return dict(case=case, P=P, Q=Q.contiguous(), d=d, out=out, res=res, seed=seed)
    target, drafters = _models(case["shape"], gen)
    g = M.MetaSD(target, drafters, gamma_max=case["gamma"], max_ctx=_max_ctx(case), temperature=case["T"], seed=seed,
                 batch=case.get("batch", 1), share_target_kv=case["shape"] in EARLY_EXIT)
    if case["prefilled"]:
        for kv in {t.data_ptr(): t for t in [g.kv_target] + g.kv_drafters}.values():
            kv.normal_(0.0, 1.0, generator=gen)
    prng = np.random.default_rng(seed)
    prompts = [prng.integers(0, target[0]["vocab"], n, dtype=np.int32) for n in _lengths(case)]
    return dict(case=case, g=g, prompts=prompts)


def run(state):
    case = state["case"]
    if case["kind"] == "accept":
        M.accept_logits(state["P"], state["Q"], state["d"], case["T"], state["seed"], out=state["out"])
        return [state["res"], state["out"]["bd"]]
    g, gamma, B = state["g"], case["gamma"], case.get("batch", 1)
    for b, prompt in enumerate(state["prompts"]):
        g.set_context(prompt, kv_prefilled=case["prefilled"], seq=b)
    steps, rewards = [], []
    for _ in range(case["rounds"]):
        if B > 1:
            ks = [g.bandit_select(seq=b) for b in range(B)]
            g.draft(ks, gamma)
            g.verify(gamma)
            n, tok, mask, bd = g.accept(gamma)
            for b in range(B):
                g.bandit_update(ks[b], int(n[b]), gamma, float(bd[b]), seq=b)
            steps.append([ks, n, tok, mask])
            rewards.append(bd)
        elif case["tree"]:
            k = g.bandit_select()
            g.draft_tree(k, TREE["parent"], TREE["rank"])
            g.verify_tree()
            n, tok, path = g.accept_tree()
            g.bandit_update(k, n, TREE["depth"])
            steps.append([k, n, tok] + path + [0] * (TREE["depth"] - len(path)))
        else:
            k, n, tok, mask, bd = g.round(gamma)
            steps.append([k, n, tok, mask])
            rewards.append(bd)
    out = [np.array(steps, np.int64), np.array(rewards, np.float64)]
    if case["kind"] == "query" and case["tree"]:
        out = [out[0], g.peek("P")[: len(TREE["parent"])]]
    elif B > 1:
        out += [g.peek("P", gamma), g.peek("Q", gamma)]
    else:
        out += [g.peek("P"), g.peek("Q")]
    if B == 1:
        out.append(g.kv_target)                               # what the prefill and the rounds left in the cache
    return out


def _per_token(desc):
    """(bytes of the weights a forward reads, multiply-adds per row, bytes of K/V per position)"""
    d, H, KH, f, L = (desc[k] for k in ("d_model", "n_heads", "n_kv_heads", "d_ffn", "n_layers"))
    hd, es = d // H, 2 if desc["dtype"] == BF16 else 4
    n = L * (2 * d * H * hd + 2 * d * KH * hd + (3 if desc["act"] == SWIGLU else 2) * d * f)
    return n, desc["vocab"] * d, 2 * L * KH * hd * es, es


def work(case):
    if case["kind"] == "accept":
        values = case["rows"] * (2 * case["gamma"] + 1) * case["vocab"]
        return dict(bytes=4.0 * values + case["rows"] * (16 + 8 * case["gamma"]), flops=8.0 * values)
    gamma, rounds, ctx = case["gamma"], case["rounds"], sum(_lengths(case))
    B = case.get("batch", 1)
    rows = len(TREE["parent"]) if case.get("tree") else gamma + 1
    steps = TREE["depth"] if case.get("tree") else gamma        # forward passes of a drafter in a round
    target = TARGET[case["shape"]]
    if case["shape"] in EARLY_EXIT:
        e = EARLY_EXIT[case["shape"]]
        drafter = dict(target, n_layers=sum(e) / len(e))
    else:
        drafter = DRAFTER[case["shape"]]
    total, flops = 0.0, 0.0
    for desc, passes, m in ((target, rounds, rows), (drafter, rounds * steps, 1)):
        n, head, kv, es = _per_token(desc)
        total += passes * ((n + head) * es + kv * (ctx + B * m) + B * m * desc["vocab"] * 4)
        flops += passes * B * m * 2.0 * (n + head) + passes * m * 2.0 * ctx * 2 * desc["n_layers"] * desc["d_model"]
    if not case["prefilled"]:
        for desc in (target,) if case["shape"] in EARLY_EXIT else (target, drafter):
            n, _, kv, es = _per_token(desc)
            total += n * es + kv * ctx
            flops += 2.0 * n * ctx + sum(2.0 * l * l * desc["n_layers"] * desc["d_model"] for l in _lengths(case))
    return dict(bytes=total, flops=flops)


def tolerance(case):
    # Measured between the library's own variants of a path (other splits of the sums, other kernels), the largest over the
    # ranges above, times four: logits 1e-4 and K/V rows 6.5e-4 (an element that rounds to the other bf16 neighbour is off by
    # one ulp, 0.008), the BD terms of the accept step 4e-8 in fp32 sums.
    if case["kind"] == "accept":
        return dict(rel=1e-6, max=1e-5, differ=0.01)
    if case["shape"] == "tiny":
        return dict(rel=2e-5, max=1e-3)
    return dict(rel=3e-3, max=0.04)
