"""The work that users of this library have it do, as cases that can be prepared, run and compared.

Four kinds of pass, all through the public binding:

  stream    one layer's whole prompt, chunk by chunk (prefill): ltri_reset, then per chunk either one ltri_step or
            the three calls append, retrieve, attend. The chunk's rows come with the call or are in the arenas
            already; several sequences can share every call.
  generate  prompts of several sequences (prefill, batched) and then one token per step for all of them (ltri_step).
  decode    step 2 and step 3 for one to four new tokens of every sequence on top of a long stored context:
            ltri_retrieve with the selection copied out, then ltri_attend. (The append of the tokens is part of
            prepare, so that a pass finds the context as it was; `generate` has appends of single tokens in it.)
  gather    the standalone copy of one sequence's attended rows (initial | retrieved | window) to packed buffers.

Keys are planted spans: a mean vector per span and noise around it, span lengths drawn at random; queries and
values are normal. Attention weights over such keys are those of ordinary activations of a trained layer in scale.
"""
import math

import numpy as np
import torch

from paper_2412_04757_amd import LtriContext, config_from_workload
from paper_2412_04757_amd.binding import MAP_LOGIT, MAP_SOFTMAX, REP_DYNAMIC, REP_MEAN

DEVICE = "cuda:0"

BASE = {
    "kind": "stream", "heads_q": 32, "heads_kv": 8, "dim": 128, "dtype": "bf16", "seqs": 1,
    "tokens": 32768, "chunk": 1024, "sink": 4, "window": 4096, "k_max": 0, "budget": 4096,
    "span_lo": 16, "span_hi": 1024,          # planted span lengths, log-uniform
    "index": "mean",                         # mean | units (dynamic vectors, 128-token units) | paper (softmax map, percentile theta as well)
    "offload": False,                        # evicted rows in host memory
    "entry": "step",                         # step | calls
    "rows_passed": True,                     # the chunk's K/V rows come with the call (else they are in the arenas)
    "lse": False,
    "generate": 0,                           # generate: tokens per sequence after the prompt
    "rows": 1,                               # decode: new tokens per sequence
}


def _case(**kw):
    c = dict(BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the benchmark's stream: a 128K prompt of a Llama-3-8B-shaped layer, rows written into the arenas in place
        _case(name="stream-128k", tokens=131072, chunk=2048, budget=8192, rows_passed=False),
        # a 32K prompt in chunks of 1024, as a model's attention layer calls it: rows handed over with the call
        _case(name="stream-32k", span_lo=32, span_hi=512),
        # a prompt length and chunk that fit no tile; log-sum-exp wanted as well
        _case(name="stream-ragged", tokens=20011, chunk=700, window=1024, budget=2048, lse=True),
        # four prompts prefilled together in small chunks
        _case(name="stream-batch", seqs=4, tokens=8192, chunk=256, window=1024, budget=1024, span_hi=256),
        # fp32, the small configuration (4 query heads on one KV head, 64 wide), by the three calls
        _case(name="stream-4k-f32", heads_q=4, heads_kv=1, dim=64, dtype="f32", tokens=4096, chunk=256, window=512,
              k_max=8, budget=0, span_lo=16, span_hi=128, entry="calls"),
        # dynamic index vectors under a budget per 128-token unit, retrieval by units
        _case(name="stream-units", chunk=2048, budget=8192, index="units"),
        # the paper's settings: softmax map, 90th-percentile threshold, IoU 0.1, chunks = units of 128 tokens
        _case(name="stream-paper", tokens=8192, chunk=128, window=1024, budget=1024, span_lo=8, span_hi=48, index="paper"),
        # evicted keys and values in host memory
        _case(name="stream-offload", offload=True, span_lo=32, span_hi=512),
        # a served batch: eight prompts of 2K tokens, then 64 tokens for each
        _case(name="generate", kind="generate", seqs=8, tokens=2048, chunk=1024, window=512, budget=512, generate=64,
              span_hi=256),
        # decoding over 128K tokens of context, 16 sequences
        _case(name="decode-128k", kind="decode", seqs=16, tokens=131072, chunk=2048, window=1024, budget=4096),
        # the smallest call: one token of one sequence
        _case(name="decode-one", kind="decode", seqs=1, tokens=16384, chunk=2048, window=1024, budget=1024),
        # the concatenated context set of a 128K stream's last chunk
        _case(name="gather-128k", kind="gather", tokens=131072, chunk=2048, budget=8192),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["stream"] * 12 + ["generate"] * 3 + ["decode"] * 4 + ["gather"])
    heads_q, heads_kv = rng.choice([(32, 8)] * 5 + [(8, 8), (16, 8), (64, 8), (16, 2)])
    c = dict(kind=kind, heads_q=heads_q, heads_kv=heads_kv, window=_log_int(rng, 256, 4096), budget=_log_int(rng, 256, 8192),
             span_lo=16, span_hi=_log_int(rng, 128, 1024))
    if kind == "stream":
        index = rng.choice(["mean"] * 7 + ["units", "paper"])
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        if dtype == "f32":
            heads_q, heads_kv, dim = rng.choice([(4, 1, 64), (4, 2, 128), (8, 2, 64)])
            c.update(heads_q=heads_q, heads_kv=heads_kv, dim=dim, dtype=dtype, budget=_log_int(rng, 128, 1024),
                     window=_log_int(rng, 64, 512))
            tokens = _log_int(rng, 1024, 6000)
        else:
            tokens = _log_int(rng, 2048, 65536)
        if index == "paper":
            tokens = min(tokens, 12000)
        seqs = rng.choice([1, 1, 1, 2, 3, 4]) if tokens <= 16384 else 1
        # at most 64 chunks; from short ones to the longest the library takes
        chunk = min(tokens, _log_int(rng, max(96, tokens / 64), 2048))
        if index == "paper":
            chunk = max(128, -(-tokens // 64 // 128) * 128)
            c.update(span_lo=8, span_hi=48)
        c.update(index=index, tokens=tokens, seqs=seqs, chunk=chunk, lse=rng.random() < 0.3,
                 entry=rng.choice(["step", "step", "calls"]), rows_passed=rng.random() < 0.7,
                 offload=dtype == "bf16" and index == "mean" and rng.random() < 0.1)
        if c["offload"]:
            c["rows_passed"] = True
    elif kind == "generate":
        c.update(seqs=rng.randint(1, 16), tokens=_log_int(rng, 512, 4096), chunk=_log_int(rng, 256, 2048),
                 generate=rng.randint(24, 96), window=_log_int(rng, 128, 1024), budget=_log_int(rng, 128, 1024))
    elif kind == "decode":
        c.update(seqs=rng.randint(1, 16), tokens=_log_int(rng, 1024, 131072), chunk=2048, rows=rng.choice([1, 1, 1, 2, 3, 4]))
    else:
        c.update(tokens=_log_int(rng, 8192, 131072), chunk=2048)
    return _case(**c)


# ------------------------------------------------------------------ inputs

def _planted_keys(out, rng, gen, lo, hi):
    """Fill out [H][T][d] with planted spans, 0.3 noise around a normal mean per span."""
    H, T, d = out.shape
    for h in range(H):
        lens = []
        left = T
        while left > 0:
            n = min(int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))), left)
            lens.append(n)
            left -= n
        mu = torch.randn((len(lens), d), generator=gen, device=DEVICE)
        row = torch.from_numpy(np.repeat(np.arange(len(lens)), lens)).to(DEVICE)
        out[h].copy_(mu[row].add_(torch.randn((T, d), generator=gen, device=DEVICE), alpha=0.3))


def _normal(shape, gen, dtype):
    out = torch.empty(shape, dtype=dtype, device=DEVICE)
    flat = out.view(-1)
    step = 1 << 28
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n].copy_(torch.randn(n, generator=gen, device=DEVICE))
    return out


def _context(c, n_layers=1):
    class W:                     # the shape, in the form config_from_workload takes
        n_q_heads, n_kv_heads, head_dim, dtype = c["heads_q"], c["heads_kv"], c["dim"], c["dtype"]
        n_seqs, context = c["seqs"], c["tokens"] + c["generate"] + (c["rows"] if c["kind"] == "decode" else 0)
        n_sink, window, k_max, budget_tokens = c["sink"], c["window"], c["k_max"], c["budget"]
        chunk = c["chunk"]
    W.n_layers = n_layers
    kw = dict(seg_map=MAP_LOGIT, theta=0.5 * math.sqrt(c["dim"]), phi=0.0, rep_mode=REP_MEAN, kv_offload=int(c["offload"]))
    if c["index"] == "units":
        kw.update(rep_mode=REP_DYNAMIC, lam=3.0, unit_tokens=128, index_block_max=12)
    elif c["index"] == "paper":
        kw.update(seg_map=MAP_SOFTMAX, theta_quantile=0.9, phi=0.1, max_spans_per_chunk=4 * (c["chunk"] // 128),
                  rep_mode=REP_DYNAMIC, lam=3.0, unit_tokens=128, index_block_max=12, max_spans=W.context // 8 + 64)
    return LtriContext(config_from_workload(W, **kw), torch.device(DEVICE))


def _cuts(tokens, chunk):
    return [(c0, min(chunk, tokens - c0)) for c0 in range(0, tokens, chunk)]


def prepare(case, seed):
    c = dict(BASE)
    c.update(case)
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    S, Hq, Hk, d, T = c["seqs"], c["heads_q"], c["heads_kv"], c["dim"], c["tokens"]
    ctx = _context(c)
    st = {"kind": c["kind"], "entry": c["entry"], "ctx": ctx, "S": S}
    if c["kind"] in ("stream", "generate"):
        cuts = _cuts(T, c["chunk"]) + [(T + i, 1) for i in range(c["generate"])]
        total = T + c["generate"]
        K = torch.empty((S, Hk, total, d), dtype=dt, device=DEVICE)
        for s in range(S):
            _planted_keys(K[s], rng, gen, c["span_lo"], c["span_hi"])
        V = _normal((S, Hk, total, d), gen, dt)
        st["out"] = torch.zeros(S * total * Hq * d, dtype=dt, device=DEVICE)
        st["lse"] = torch.zeros(S * total * Hq, dtype=torch.float32, device=DEVICE) if c["lse"] else None
        Q = _normal((S * total * Hq * d,), gen, dt)
        if not c["rows_passed"]:
            ka, va = ctx.arena_views()
            ka[0].copy_(K)
            va[0].copy_(V)
        chunks, at = [], 0
        for c0, n in cuts:
            m = S * n * Hq
            k = K[:, :, c0:c0 + n].contiguous() if c["rows_passed"] else None
            v = V[:, :, c0:c0 + n].contiguous() if c["rows_passed"] else None
            chunks.append((n, k, v, Q[at * d:(at + m) * d].view(S, n, Hq, d), st["out"][at * d:(at + m) * d].view(S, n, Hq, d),
                           st["lse"][at:at + m].view(S, n, Hq) if c["lse"] else None))
            at += m
        st["chunks"] = chunks
        return st
    # decode, gather: the context is stored and indexed beforehand
    extra = c["rows"] if c["kind"] == "decode" else 0
    ka, va = ctx.arena_views()
    for s in range(S):
        _planted_keys(ka[0, s], rng, gen, c["span_lo"], c["span_hi"])
        va[0, s].copy_(_normal(va[0, s].shape, gen, dt))
    if c["kind"] == "decode":
        for c0, n in _cuts(T, c["chunk"]):
            ctx.append_chunk(0, 0, S, n)
        ctx.append_chunk(0, 0, S, extra)
        st["q"] = _normal((S, extra, Hq, d), gen, dt)
        st["out"] = torch.zeros((S, extra, Hq, d), dtype=dt, device=DEVICE)
        st["ids"] = torch.full((S, Hk, ctx.sel_cap), -1, dtype=torch.int32, device=DEVICE)
        st["cnt"] = torch.zeros((S, Hk), dtype=torch.int32, device=DEVICE)
    else:
        cuts = _cuts(T, c["chunk"])
        for c0, n in cuts:
            ctx.append_chunk(0, 0, 1, n)
        ctx.retrieve(0, 0, 1, _normal((1, cuts[-1][1], Hq, d), gen, dt))
        st["k"] = torch.zeros((Hk, ctx.list_cap, d), dtype=dt, device=DEVICE)
        st["v"] = torch.zeros((Hk, ctx.list_cap, d), dtype=dt, device=DEVICE)
        st["n"] = torch.zeros((Hk,), dtype=torch.int32, device=DEVICE)
    if ctx.sync_status() != 0:
        raise RuntimeError("the context could not be stored")
    return st


# ------------------------------------------------------------------ one pass

def run(st):
    ctx, S = st["ctx"], st["S"]
    if st["kind"] in ("stream", "generate"):
        for s in range(S):
            ctx.reset(s)
        if st["entry"] == "step":
            for n, k, v, q, out, lse in st["chunks"]:
                ctx.step(0, 0, S, k, v, q, out=out, lse=lse)
        else:
            for n, k, v, q, out, lse in st["chunks"]:
                ctx.append_chunk(0, 0, S, n, k_chunk=k, v_chunk=v)
                ctx.retrieve(0, 0, S, q)
                ctx.attend(0, 0, S, q, out=out, lse=lse)
        return {"out": st["out"], "lse": st["lse"]}
    if st["kind"] == "decode":
        ctx.retrieve(0, 0, S, st["q"], sel_ids=st["ids"], sel_cnt=st["cnt"])
        ctx.attend(0, 0, S, st["q"], out=st["out"])
        return {"out": st["out"], "cnt": st["cnt"], "ids": st["ids"]}
    ctx.gather_pack(0, 0, st["k"], st["v"], st["n"])
    return {"k": st["k"], "v": st["v"], "n": st["n"]}


# ------------------------------------------------------------------ what a pass cannot do without

def _attended(c, c0):
    """Context tokens of a chunk that starts at c0: initial, retrieved (by the budget or the count), window."""
    mean = (c["span_hi"] - c["span_lo"]) / math.log(c["span_hi"] / c["span_lo"])
    retrieved = c["budget"] or c["k_max"] * mean
    return min(c0, c["sink"] + c["window"] + retrieved)


def work(case):
    c = dict(BASE)
    c.update(case)
    S, Hq, Hk, d = c["seqs"], c["heads_q"], c["heads_kv"], c["dim"]
    elt = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "gather":
        return {"bytes": 2 * 2 * Hk * _attended(c, c["tokens"]) * d * elt, "flops": 0}
    if c["kind"] == "decode":
        n, rows = _attended(c, c["tokens"]), c["rows"]
        spans = c["tokens"] * math.log(c["span_hi"] / c["span_lo"]) / (c["span_hi"] - c["span_lo"])
        return {"bytes": S * (2 * Hk * (n + rows) * d * elt + Hk * spans * d * elt + 2 * rows * Hq * d * elt),
                "flops": S * Hq * 4 * d * rows * (n + (rows + 1) / 2)}
    flops, nbytes = 0.0, 0.0
    for c0, n in _cuts(c["tokens"], c["chunk"]) + [(c["tokens"] + i, 1) for i in range(c["generate"])]:
        flops += S * Hq * 4 * d * n * (_attended(c, c0) + (n + 1) / 2)
        flops += S * Hk * d * n * (n + 1)                       # the chunk's own causal map, once
        nbytes += S * (2 * Hk + 2 * Hq) * n * d * elt
        if n == 1:                                              # a single token's step has to read its context
            nbytes += S * 2 * Hk * _attended(c, c0) * d * elt
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    c = dict(BASE)
    c.update(case)
    if c["kind"] == "gather":
        return "exact"
    # the probabilities and the output are rounded to bf16 (fp32: the sums are); selections are whole numbers and agree
    return {"rel": 1e-5} if c["dtype"] == "f32" else {"rel": 1e-2}
