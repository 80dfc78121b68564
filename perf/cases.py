"""Measured cases of the verification step: what a user of this library has it do, through its
public entry points, over the range of sizes it serves.

  wisp_verify          whole calls on the Llama-3-8B and -70B shapes cut to a few layers (every
                       kernel at the full widths and row counts of the served batches) and on
                       the small fp32 model: single sessions, batches of follow-ups, first-time
                       verifications of long prompts, alone and mixed with follow-ups
  wisp_attention       one layer's ragged paged attention
  wisp_accept          the acceptance alone, on given logits
  wisp_draft_stats     the draft-side statistics
  wisp_reject_predict  the draft-side predictor

The models are cut in depth because bf16 rounding differences grow from layer to layer: a whole
32-layer model would not show more of the path, only more of that.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2601_11652_amd as W

PAGE = 16
# layers, d_model, query heads, kv heads, head_dim, d_ff, vocab, storage, rotary base
SHAPES = {
    "tiny": (2, 256, 4, 4, 64, 1024, 1024, "f32", 1e4),
    "8b": (4, 4096, 32, 8, 128, 14336, 128256, "bf16", 5e5),
    "70b": (2, 8192, 64, 8, 128, 28672, 128256, "bf16", 5e5),
}
WEIGHT_STD = 0.02
KV_STD = 1.15          # what projections of unit-RMS rows by such weights give at d = 4096


class Shape:
    """The attributes of a model shape that GpuModel reads."""

    def __init__(self, key: str):
        (self.n_layers, self.d_model, self.n_q_heads, self.n_kv_heads, self.head_dim, self.d_ff, self.vocab,
         self.dtype, self.rope_base) = SHAPES[key]
        self.name, self.rms_eps = key, 1e-5
        self.es = 4 if self.dtype == "f32" else 2
        self.torch = torch.float32 if self.dtype == "f32" else torch.bfloat16
        self.group = self.n_q_heads // self.n_kv_heads
        self.layer_params = self.d_model * ((2 * self.n_q_heads + 2 * self.n_kv_heads) * self.head_dim + 3 * self.d_ff)


# ------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------
def _verify(name, shape, requests, ctx, gamma, cold=0, prompt=(0, 0), mix=1, log=True):
    """`requests` follow-ups with cached contexts drawn from ctx (log-uniform or uniform) and
    drafts from gamma, after `cold` first-time requests whose prompts are drawn from `prompt`."""
    return dict(name=name, kind="verify", shape=shape, requests=requests, ctx_lo=ctx[0], ctx_hi=ctx[1], ctx_log=log,
                gamma_lo=gamma[0], gamma_hi=gamma[1], plain=0.0, cold=cold, prompt_lo=prompt[0],
                prompt_hi=prompt[1], mix=mix)


def _attention(name, shape, requests, ctx, gamma, plain=0.0, mix=1, log=True):
    return dict(_verify(name, shape, requests, ctx, gamma, mix=mix, log=log), kind="attention", plain=plain)


def listed():
    return [
        # the small fp32 model that the parity and session checks serve: launches and latency
        _verify("verify_tiny_f32", "tiny", 4, (32, 128), (1, 4), log=False),
        # one session in a chat, the least a server verifies at a time
        _verify("verify_8b_b1", "8b", 1, (1300, 1300), (5, 5)),
        # the benchmark's headline batch: 32 sessions of 512-2048 cached tokens
        _verify("verify_8b_b32", "8b", 32, (512, 2048), (1, 8), mix=18, log=False),
        # a loaded server: 256 sessions of 1024-8192 cached tokens
        _verify("verify_8b_b256", "8b", 256, (1024, 8192), (2, 6), mix=1),
        # the large model's batch
        _verify("verify_70b_b64", "70b", 64, (1024, 4096), (1, 8), mix=52, log=False),
        # a long prompt's first verification with one short follow-up caught in its batch
        _verify("prefill_8b_4096", "8b", 1, (500, 500), (5, 5), cold=1, prompt=(4096, 4096)),
        # a few new sessions' prompts among the follow-ups of running ones
        _verify("prefill_8b_mixed", "8b", 24, (128, 3072), (1, 5), cold=3, prompt=(64, 512)),
        # one layer's attention for the headline batch
        _attention("attention_8b_b32", "8b", 32, (512, 2048), (1, 8), mix=18, log=False),
        # one layer's attention for contexts of very different lengths, a quarter plain decoding
        _attention("attention_8b_dyn128", "8b", 128, (256, 32768), (1, 16), plain=0.25),
        # the acceptance on logits that come from elsewhere
        dict(name="accept_b32", kind="accept", requests=32, gamma_lo=1, gamma_hi=8, vocab=128256, temperature=1.0, mix=18),
        # a draft server's statistics for the tokens that its sessions just drafted
        dict(name="draft_stats_256", kind="stats", rows=256, vocab=128256, temperature=0.8),
        # the predictor on those of a small batch
        dict(name="reject_predict_32", kind="predict", rows=32, n_in=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["verify", "verify70", "prefill", "tiny", "attention", "accept", "stats", "predict"],
                       [6, 2, 3, 1, 3, 2, 1, 1])[0]
    mix = rng.randrange(1, 1 << 30)
    if kind in ("verify", "verify70", "attention"):
        big = 64 if kind == "verify70" else 256
        n = _log_int(rng, 1, big)
        hi = _log_int(rng, 256, min(32768 if kind == "attention" else 8192, (700 if kind != "verify70" else 128) * 1024 // n))
        lo = max(1, int(hi * rng.uniform(0.05, 1.0)))
        g_hi = rng.randint(1, max(1, min(8 if kind != "attention" else 16, (2200 if big == 256 else 660) // n - 1)))
        g_lo = rng.randint(0, g_hi)
        if kind == "attention":
            c = _attention("", "8b", n, (lo, hi), (g_lo, g_hi), plain=rng.choice([0.0, 0.25]), mix=mix)
        else:
            c = _verify("", "8b" if kind == "verify" else "70b", n, (lo, hi), (g_lo, g_hi), mix=mix,
                        log=rng.random() < 0.5)
    elif kind == "prefill":
        cold = rng.randint(1, 4)
        hi = _log_int(rng, 64, 4096 // cold)
        n = rng.randint(0, 16)
        c = _verify("", "8b", n, (64, _log_int(rng, 128, 3072)), (0, rng.randint(1, 5)), cold=cold,
                    prompt=(max(1, int(hi * rng.uniform(0.1, 1.0))), hi), mix=mix)
    elif kind == "tiny":
        c = _verify("", "tiny", _log_int(rng, 1, 32), (1, _log_int(rng, 32, 512)), (0, rng.randint(1, 8)), mix=mix)
    elif kind == "accept":
        n = _log_int(rng, 1, 192)
        c = dict(kind="accept", requests=n, gamma_lo=0, gamma_hi=rng.randint(1, min(16, 1800 // n)),
                 vocab=rng.choice([128256, 128256, 32000, rng.randint(1000, 150000)]),
                 temperature=rng.choice([1.0, 1.0, 0.6, 0.0]), mix=mix)
    elif kind == "stats":
        c = dict(kind="stats", rows=_log_int(rng, 1, 1024), vocab=rng.choice([128256, 32000, rng.randint(1000, 150000)]),
                 temperature=round(rng.uniform(0.7, 1.3), 2))
    else:
        c = dict(kind="predict", rows=_log_int(rng, 1, 1024), n_in=rng.choice([4, 5]))
    c.pop("name", None)
    return c


def _lengths(case):
    """(cached context, prompt rows, drafts) of each request, from the case alone."""
    r = np.random.default_rng([case["mix"], 2601])

    def log_ints(lo, hi, n):
        return np.clip(np.rint(np.exp(r.uniform(math.log(lo), math.log(hi), n))), lo, hi).astype(np.int32)

    n, cold = case["requests"], case.get("cold", 0)
    gam = r.integers(case["gamma_lo"], case["gamma_hi"], n + cold, endpoint=True).astype(np.int32)
    gam = np.where(r.random(n + cold) < case.get("plain", 0.0), 0, gam).astype(np.int32)
    ctx, pre = np.zeros(n + cold, np.int32), np.zeros(n + cold, np.int32)
    if "ctx_lo" in case:
        if case["ctx_log"]:
            ctx[cold:] = log_ints(case["ctx_lo"], case["ctx_hi"], n)
        else:
            ctx[cold:] = r.integers(case["ctx_lo"], case["ctx_hi"], n, endpoint=True)
        if cold:
            pre[:cold] = log_ints(case["prompt_lo"], case["prompt_hi"], cold)
    return ctx, pre, gam


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
def _gen(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + tag) & ((1 << 62) - 1))
    return g


def _normal(shape, std, dtype, g):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)


def _layer(s, seed, l):
    """Layer l's weights in their natural [out][in] layout."""
    g = _gen(seed, 100 + l)
    q, kv = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    dims = {"wq": (q, s.d_model), "wk": (kv, s.d_model), "wv": (kv, s.d_model), "wo": (s.d_model, q),
            "w_gate": (s.d_ff, s.d_model), "w_up": (s.d_ff, s.d_model), "w_down": (s.d_model, s.d_ff)}
    w = {k: _normal(v, WEIGHT_STD, s.torch, g) for k, v in dims.items()}
    for k in ("attn_norm", "mlp_norm"):
        w[k] = (1.0 + 0.1 * torch.randn(s.d_model, device="cuda", generator=g)).to(s.torch)
    return w


def _globals(s, seed):
    g = _gen(seed, 1)
    return {"embed": _normal((s.vocab, s.d_model), WEIGHT_STD, s.torch, g),
            "lm_head": _normal((s.vocab, s.d_model), WEIGHT_STD, s.torch, g),
            "final_norm": (1.0 + 0.1 * torch.randn(s.d_model, device="cuda", generator=g)).to(s.torch)}


def _page_table(tokens, seed):
    """Scattered pages: a permutation of the pool, -1 past a request's last page."""
    need = (tokens.astype(np.int64) + PAGE - 1) // PAGE
    n_blocks = int(need.sum()) + 3
    perm = np.random.default_rng([int(seed), 7]).permutation(n_blocks).astype(np.int32)
    tab = np.full((len(need), int(need.max())), -1, np.int32)
    o = 0
    for i, k in enumerate(need):
        tab[i, :k] = perm[o:o + k]
        o += k
    return tab, n_blocks


def _pools(s, layers, n_blocks, seed):
    g = _gen(seed, 2)
    shp = (layers, n_blocks, s.n_kv_heads, PAGE * s.head_dim)
    return _normal(shp, KV_STD, s.torch, g), _normal(shp, KV_STD, s.torch, g)


def _drafts(n, vocab, g):
    """Draft distributions q (peaked, as a language model's) and a token drawn from each."""
    q = torch.empty(max(n, 1), vocab, device="cuda")
    y = torch.empty(max(n, 1), dtype=torch.int64, device="cuda")
    for a in range(0, n, 256):
        b = min(n, a + 256)
        q[a:b] = torch.softmax(2.5 * torch.randn(b - a, vocab, device="cuda", generator=g), -1)
        y[a:b] = torch.multinomial(q[a:b], 1, generator=g)[:, 0]
    return q, y[:n]


def _prepare_step(case, seed):
    s = Shape(case["shape"])
    ctx, pre, gam = _lengths(case)
    tab, n_blocks = _page_table(ctx + pre + gam + 1, seed)
    pt = torch.as_tensor(tab, device="cuda")
    attn = case["kind"] == "attention"
    kv = W.KVPool(*_pools(s, 1 if attn else s.n_layers, n_blocks, seed))
    desc = W.BatchDesc(ctx, gam, pt, 1.0, None, pre if pre.any() else None)
    if attn:
        model = W.GpuModel.shape_only(s)
        q = _normal((desc.rows, s.n_q_heads, s.head_dim), 1.15, s.torch, _gen(seed, 3))
        return dict(kind="attention", model=model, kv=kv, desc=desc, q=q, out=torch.empty_like(q),
                    ws=W.workspace(W.wisp_workspace_size(model, desc)))
    gm = W.GpuModel(s, lambda l: _layer(s, seed, l), _globals(s, seed))
    g = _gen(seed, 4)
    q, y = _drafts(desc.S, s.vocab, g)
    tokens = torch.randint(0, s.vocab, (desc.rows,), device="cuda", dtype=torch.int32, generator=g)
    first = np.cumsum(pre + gam + 1) - gam           # the first draft's row of each request
    at = np.concatenate([np.arange(f, f + k) for f, k in zip(first, gam)]) if desc.S else np.zeros(0)
    tokens[torch.as_tensor(at.astype(np.int64), device="cuda")] = y.to(torch.int32)
    return dict(kind="verify", gm=gm, kv=kv, desc=desc, tokens=tokens, q=q, seed=int(seed) + 77,
                acc=torch.empty(desc.B, dtype=torch.int32, device="cuda"),
                out=torch.empty(desc.M, dtype=torch.int32, device="cuda"),
                logits=torch.empty(desc.M, s.vocab, device="cuda"),
                ws=W.workspace(W.wisp_workspace_size(gm.c, desc)), decisions=s.dtype == "f32")


def _prepare_accept(case, seed):
    """Target logits near the drafts' own (a draft model that mostly agrees with its target)."""
    _, _, gam = _lengths(case)
    desc = W.BatchDesc(np.zeros_like(gam), gam, None, case["temperature"])
    V, g = case["vocab"], _gen(seed, 5)
    logits = 2.5 * torch.randn(desc.M, V, device="cuda", generator=g)
    last = np.cumsum(gam + 1) - 1
    rows = np.setdiff1d(np.arange(desc.M), last)     # the rows that score a draft
    q = torch.empty(max(desc.S, 1), V, device="cuda")
    tokens = torch.randint(0, V, (desc.M,), device="cuda", dtype=torch.int32, generator=g)
    for a in range(0, desc.S, 256):
        r = torch.as_tensor(rows[a:a + 256], device="cuda")
        q[a:a + len(r)] = torch.softmax(logits[r] + 0.5 * torch.randn(len(r), V, device="cuda", generator=g), -1)
        tokens[r + 1] = torch.multinomial(q[a:a + len(r)], 1, generator=g)[:, 0].to(torch.int32)
    return dict(kind="accept", desc=desc, vocab=V, logits=logits, tokens=tokens, q=q, seed=int(seed) + 78,
                acc=torch.empty(desc.B, dtype=torch.int32, device="cuda"),
                out=torch.empty(desc.M, dtype=torch.int32, device="cuda"),
                ws=W.workspace(W.wisp_accept_workspace_size(desc, V)))


def _stats_logits(case, seed):
    return 2.5 * torch.randn(case["rows"], case["vocab"], device="cuda", generator=_gen(seed, 6)) + 0.5


def _mlp(case, seed):
    g, n = _gen(seed, 7), case["n_in"]

    def r(*shape):
        return torch.randn(*shape, device="cuda", generator=g)

    p = {"mean": 0.5 * r(n), "inv_std": 1.0 + r(n).abs(), "w1": r(512, n) / 2, "b1": 0.1 * r(512),
         "w2": r(128, 512) / 16, "b2": 0.1 * r(128), "w3": r(64, 128) / 8, "b3": 0.1 * r(64), "w4": r(64) / 8,
         "b4": 0.1}
    return p, r(case["rows"], n)


def prepare(case, seed):
    if case["kind"] in ("verify", "attention"):
        return _prepare_step(case, seed)
    if case["kind"] == "accept":
        return _prepare_accept(case, seed)
    if case["kind"] == "stats":
        x = _stats_logits(case, seed)
        n = W.lib.wisp_draft_stats_workspace_size(case["rows"], case["vocab"])
        return dict(kind="stats", x=x, vocab=case["vocab"], T=case["temperature"], ws=W.workspace(n),
                    stats=torch.empty(case["rows"], 4, device="cuda"))
    p, f = _mlp(case, seed)
    return dict(kind="predict", mlp=W.RejectMLP(p), f=f, p=torch.empty(case["rows"], device="cuda"))


# ------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------
def run(st):
    if st["kind"] == "verify":
        W.wisp_verify(st["gm"].c, st["kv"], st["desc"], st["tokens"], st["q"], st["seed"], st["acc"], st["out"],
                      st["logits"], st["ws"])
        r = {"logits": st["logits"], "k": st["kv"].k, "v": st["kv"].v}
        # the draws that decide the tokens turn on the last bits of bf16 logits, so the tokens of
        # a bf16 call are compared on given logits (wisp_accept); in fp32 they come along
        if st["decisions"]:
            r.update(accept_len=st["acc"], tokens=st["out"])
        return r
    if st["kind"] == "attention":
        W.wisp_attention(st["model"], st["kv"], st["desc"], st["q"], st["out"], st["ws"])
        return st["out"]
    if st["kind"] == "accept":
        W.wisp_accept(st["desc"], st["vocab"], st["logits"], st["tokens"], st["q"], st["seed"], st["acc"], st["out"],
                      st["ws"])
        return {"accept_len": st["acc"], "tokens": st["out"]}
    if st["kind"] == "stats":
        W.wisp_draft_stats(st["x"], st["vocab"], st["T"], st["stats"], st["ws"])
        return st["stats"]
    W.wisp_reject_predict(st["mlp"], st["f"], st["p"])
    return st["p"]


def work(case):
    """Weights, cached K and V, inputs and results once; products with the rows that exist."""
    k = case["kind"]
    if k == "stats":
        n = case["rows"] * case["vocab"]
        return {"bytes": 4 * n + 16 * case["rows"], "flops": 10 * n}
    if k == "predict":
        per = 512 * case["n_in"] + 512 * 128 + 128 * 64 + 64
        return {"bytes": 4 * (per + case["rows"] * (case["n_in"] + 1)), "flops": 2 * per * case["rows"]}
    ctx, pre, gam = (x.astype(np.int64) for x in _lengths(case))
    mv = int((gam + 1).sum())
    if k == "accept":
        # every logits row once, and the q row of about half the requests (a rejection)
        v = case["vocab"]
        return {"bytes": 4 * v * (mv + len(gam) // 2), "flops": 4 * v * mv}
    s = Shape(case["shape"])
    new = pre + gam + 1
    m, kvw = int(new.sum()), s.n_kv_heads * s.head_dim * 2 * s.es
    pairs = int((new * ctx + new * (new + 1) // 2).sum())
    attn_flops = 4 * s.n_q_heads * s.head_dim * pairs
    qo = 2 * m * s.n_q_heads * s.head_dim * s.es
    if k == "attention":
        return {"bytes": int((ctx + new).sum()) * kvw + qo, "flops": attn_flops}
    n_bytes = (s.n_layers * s.layer_params + s.vocab * s.d_model) * s.es + m * s.d_model * s.es
    n_bytes += s.n_layers * int((ctx + new).sum()) * kvw + mv * s.vocab * 4 + int((gam > 0).sum()) // 2 * s.vocab * 4
    flops = s.n_layers * (2 * m * s.layer_params + attn_flops) + 2 * mv * s.vocab * s.d_model
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    k = case["kind"]
    if k == "accept":
        return "exact"                       # tokens and lengths
    if k == "stats":
        return {"rel": 1e-6, "max": 1e-5}      # 3.6e-8 from 64 bits
    if k == "predict":
        return {"rel": 1e-6, "max": 1e-5}      # 1e-7 from 64 bits
    if k == "attention":
        return {"rel": 1e-2, "max": 0.1}       # 2.3e-3 from 64 bits: bf16 probabilities and outputs
    if case["shape"] == "tiny":
        return {"rel": 4e-6, "max": 4e-5, "differ": 0.0}   # 7.6e-7 from 64 bits
    return {"rel": 0.03, "max": 0.3}         # logits 1.1e-2 to 1.4e-2 from 64 bits: bf16 layer inputs


# ------------------------------------------------------------------------------------------
# the same in 64 bits
# ------------------------------------------------------------------------------------------
def _page_index(hd):
    """Position of (slot, dim) inside a K page and a V page (the page layouts of the C ABI)."""
    s, e = np.arange(PAGE)[:, None], np.arange(hd)[None, :]
    k = (((e // 32) * 2 + (s // 4) % 2) * 4 + (e % 32) // 8) * 64 + ((s // 8) * 4 + s % 4) * 8 + e % 8
    v = ((e // 16) * 2 + s // 8) * 128 + (e % 16) * 8 + s % 8
    return torch.as_tensor(k, device="cuda"), torch.as_tensor(v, device="cuda")


def _attend(s, q, k, v, ctx):
    """q [rows][heads][hd] at positions ctx .. over k, v [tokens][kv heads][hd]."""
    rows, out = q.shape[0], torch.empty_like(q)
    for a in range(0, rows, 512):
        n = min(512, rows - a)
        keep = torch.arange(k.shape[0], device="cuda")[None, :] <= ctx + a + torch.arange(n, device="cuda")[:, None]
        for h in range(s.n_kv_heads):
            qh = q[a:a + n, h * s.group:(h + 1) * s.group].reshape(n * s.group, -1)
            sc = (qh @ k[:, h].t().contiguous()) / math.sqrt(s.head_dim)
            sc = sc.masked_fill(~keep.repeat_interleave(s.group, 0), -math.inf)
            out[a:a + n, h * s.group:(h + 1) * s.group] = (torch.softmax(sc, -1) @ v[:, h].contiguous()).reshape(n, s.group, -1)
    return out


def _exact_step(case, seed):
    s = Shape(case["shape"])
    ctx, pre, gam = _lengths(case)
    new = pre + gam + 1
    tab, n_blocks = _page_table(ctx + new, seed)
    attn = case["kind"] == "attention"
    kp, vp = _pools(s, 1 if attn else s.n_layers, n_blocks, seed)
    ki, vi = _page_index(s.head_dim)
    off = np.concatenate([[0], np.cumsum(new)])
    f64 = torch.float64

    def cached(l, i):
        """Request i's K and V [tokens][kv heads][hd] of layer l, and its page ids."""
        pages = torch.as_tensor(tab[i][tab[i] >= 0].astype(np.int64), device="cuda")

        def one(pool, idx):
            return pool[l][pages].to(f64)[:, :, idx].permute(0, 2, 1, 3).reshape(-1, s.n_kv_heads, s.head_dim)

        return one(kp, ki), one(vp, vi), pages

    if attn:
        q = _normal((int(off[-1]), s.n_q_heads, s.head_dim), 1.15, s.torch, _gen(seed, 3)).to(f64)
        return torch.cat([_attend(s, q[off[i]:off[i + 1]], *[x[:ctx[i] + new[i]] for x in cached(0, i)[:2]], int(ctx[i]))
                          for i in range(len(new))])
    tokens = _prepare_tokens(case, seed, s, ctx, pre, gam)
    pools_too = kp.numel() < 1 << 28                 # larger pools in 64 bits would not fit beside the rest
    k64, v64 = (kp.to(f64), vp.to(f64)) if pools_too else (None, None)
    glob = _globals(s, seed)
    h = glob["embed"][tokens.long()].to(f64)
    pos = torch.as_tensor(np.concatenate([np.arange(c, c + n) for c, n in zip(ctx, new)]), device="cuda", dtype=f64)
    half = s.head_dim // 2
    ang = pos[:, None] * s.rope_base ** (-2.0 * torch.arange(half, device="cuda", dtype=f64) / s.head_dim)[None, :]
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def norm(x, gain):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * gain.to(f64)

    def rope(x):
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    def linear(x, w):
        return torch.cat([x @ w[a:a + 16384].to(f64).t().contiguous() for a in range(0, w.shape[0], 16384)], -1)

    for l in range(s.n_layers):
        w = _layer(s, seed, l)
        x = norm(h, w["attn_norm"])
        q = rope(linear(x, w["wq"]).view(-1, s.n_q_heads, s.head_dim))
        k = rope(linear(x, w["wk"]).view(-1, s.n_kv_heads, s.head_dim))
        v = linear(x, w["wv"]).view(-1, s.n_kv_heads, s.head_dim)
        ao = torch.empty_like(q)
        for i in range(len(new)):
            kc, vc, pages = cached(l, i)
            a, b = int(off[i]), int(off[i + 1])
            n = int(ctx[i] + new[i])
            kc[ctx[i]:n], vc[ctx[i]:n] = k[a:b], v[a:b]
            ao[a:b] = _attend(s, q[a:b], kc[:n], vc[:n], int(ctx[i]))
            if pools_too:
                for pool, idx, x64 in ((k64, ki, kc), (v64, vi, vc)):
                    back = torch.empty(len(pages), s.n_kv_heads, PAGE * s.head_dim, device="cuda", dtype=f64)
                    back[:, :, idx] = x64.reshape(-1, PAGE, s.n_kv_heads, s.head_dim).permute(0, 2, 1, 3)
                    pool[l][pages] = back
        h = h + linear(ao.reshape(h.shape[0], -1), w["wo"])
        x = norm(h, w["mlp_norm"])
        h = h + linear(torch.nn.functional.silu(linear(x, w["w_gate"])) * linear(x, w["w_up"]), w["w_down"])
    rows = np.concatenate([np.arange(off[i + 1] - gam[i] - 1, off[i + 1]) for i in range(len(new))])
    logits = linear(norm(h[torch.as_tensor(rows, device="cuda")], glob["final_norm"]), glob["lm_head"])
    r = {"logits": logits, "k": k64, "v": v64}
    if s.dtype == "f32":
        r.update(accept_len=None, tokens=None)
    return r


def _prepare_tokens(case, seed, s, ctx, pre, gam):
    """The token ids that _prepare_step gives the call."""
    g, n = _gen(seed, 4), int(gam.sum())
    _, y = _drafts(n, s.vocab, g)
    tokens = torch.randint(0, s.vocab, (int((pre + gam + 1).sum()),), device="cuda", dtype=torch.int32, generator=g)
    first = np.cumsum(pre + gam + 1) - gam
    if n:
        at = np.concatenate([np.arange(f, f + k) for f, k in zip(first, gam)])
        tokens[torch.as_tensor(at.astype(np.int64), device="cuda")] = y.to(torch.int32)
    return tokens


def exact(case, seed):
    k = case["kind"]
    if k in ("verify", "attention"):
        return _exact_step(case, seed)
    if k == "stats":
        out = []
        for x in _stats_logits(case, seed).split(64):
            z = x.double() / case["temperature"]
            p = torch.softmax(z, -1)
            top = torch.topk(p, 2, -1).values
            ent = torch.logsumexp(z, -1) - (p * z).sum(-1)
            out.append(torch.stack([top[:, 0], ent, top[:, 0] - top[:, 1], z.std(-1, unbiased=False)], -1))
        return torch.cat(out)
    if k == "predict":
        p, f = _mlp(case, seed)
        p = {n: v.double() if isinstance(v, torch.Tensor) else v for n, v in p.items()}
        x = (f.double() - p["mean"]) * p["inv_std"]
        for w, b in (("w1", "b1"), ("w2", "b2"), ("w3", "b3")):
            x = torch.relu(x @ p[w].t().contiguous() + p[b])
        return torch.sigmoid(x @ p["w4"] + p["b4"])
    return None                              # the acceptance returns whole numbers
