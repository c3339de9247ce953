"""Which spans step 2 selects, at the span counts where its kernels change method. Keys and queries are whole multiples
of powers of two, so every score is exact and ties are real ties."""
import numpy as np
import pytest
import torch

from paper_2412_04757_amd import LtriContext, config_from_workload
from workloads import Workload

pytestmark = pytest.mark.gpu

SINK, WINDOW, CHUNK = 3, 37, 256


def select_reference(scores, clip, k_max, budget):
    """Ascending ids of the longest prefix, in the order (score descending, id ascending) over the spans with evicted
    tokens, within k_max spans and budget tokens (0: no limit)."""
    order = sorted((i for i in range(len(scores)) if clip[i] > 0), key=lambda i: (-scores[i], i))
    out, cum = [], 0
    for r, i in enumerate(order):
        cum += clip[i]
        if (k_max and r >= k_max) or (budget and cum > budget):
            break
        out.append(i)
    return sorted(out)


def span_values(kind, n, rng):
    """One value per span; a span's score is a fixed positive multiple of it."""
    if kind == "spread":
        return (1 + rng.integers(0, 128, n) / 128) * 2.0 ** rng.integers(-6, 7, n) * rng.choice([-1, 1], n)
    if kind == "tied":
        return np.full(n, -1.5)
    if kind == "outlier":                            # one score takes the whole range, the others share a piece of it
        v = 1 + rng.integers(0, 4, n) / 128
        v[n // 2] = 2.0 ** 30
        return v
    v = np.zeros(n)                                  # "wide": beyond fp32 on one side, tiny and zero on the other
    v[::3] = rng.choice([2.0 ** 120, -2.0 ** 120, 2.0 ** -120, -2.0 ** -120], len(v[::3]))
    return v


@pytest.mark.parametrize("dtype,kind", [("bf16", "spread"), ("bf16", "tied"), ("bf16", "outlier"), ("bf16", "wide"),
                                        ("f32", "spread"), ("f32", "wide")])
@pytest.mark.parametrize("n_spans", [1, 63, 64, 129, 256, 257, 700, 1024, 1025, 2300])
def test_selection_around_its_method_changes(gpu_device, dtype, kind, n_spans):
    """Up to 256 spans every span is compared with all others, more go by pieces of the score range, and equal or
    not representable scores by sorting. One query token and a chunk of queries, spans of 1 to 3 tokens, limits that
    bind in count, in tokens, in both and not at all."""
    rng = np.random.default_rng(n_spans)
    lens = rng.integers(1, 4, n_spans)
    total = int(lens.sum())
    T = total + WINDOW + CHUNK + 8
    sign = torch.from_numpy(rng.choice([-1.0, 1.0], 128))
    val = span_values(kind, n_spans, rng)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    scale = 2.0 ** 7 if kind == "wide" else 1.0
    rows = torch.from_numpy(np.repeat(val, lens))[:, None] * sign[None, :]
    for k_max, budget in ((7, 0), (0, max(3, total // 3)), (n_spans // 2 + 1, total // 4 + 2), (0, T)):
        w = Workload("mini-select", 4, 1, 128, dtype, T, CHUNK, SINK, WINDOW, k_max, budget, "uniform", 16, 128)
        ctx = LtriContext(config_from_workload(w, n_layers=1, max_tokens=T, theta=1e30, max_spans=n_spans + 64), gpu_device)
        ka, va = ctx.arena_views()
        ka.zero_(), va.zero_()
        ka[0, 0, 0, :total].copy_(rows.to(dt))
        for one_token in (True, False):
            ctx.reset(0)
            at = 0
            while at < n_spans:                      # whole spans per chunk, at most CHUNK tokens
                cum = np.cumsum(lens[at:])
                k = int(np.searchsorted(cum, CHUNK, side="right"))
                ctx.append_chunk_with_spans(0, 0, int(cum[k - 1]), [np.concatenate([[0], cum[:k]])])
                at += k
            ctx.append_chunk_with_spans(0, 0, WINDOW, [np.array([0, WINDOW])])
            n = 1 if one_token else CHUNK
            if one_token:
                ctx.append_chunk(0, 0, 1, 1)
            else:
                ctx.append_chunk_with_spans(0, 0, n, [np.array([0, n])])
            q = (sign * scale).to(dt).to(gpu_device).expand(1, n, 4, 128).contiguous()
            ctx.retrieve(0, 0, 1, q)
            start = np.concatenate([[0], np.cumsum(lens)[:-1]])
            clip = np.maximum(start + lens - np.maximum(start, SINK), 0)
            want = select_reference(val, clip, k_max, budget)
            ids, _ = ctx.get_selection(0, 0, 0)
            assert list(ids) == want, (k_max, budget, one_token)
            tokens = [t for i in want for t in range(max(start[i], SINK), start[i] + lens[i])]
            here = total + WINDOW
            listed = list(range(min(SINK, here))) + tokens + list(range(max(SINK, here - WINDOW), here))
            assert list(ctx.get_token_list(0, 0, 0)) == listed
        assert ctx.sync_status() == 0


@pytest.mark.parametrize("kind", ["spread", "tied", "outlier"])
@pytest.mark.parametrize("n_units", [63, 256, 257, 1025, 2300])
def test_selection_of_memory_units(gpu_device, kind, n_units):
    """The same with units (of one token, so that a unit's score is its token's): the selection runs over unit ids."""
    rng = np.random.default_rng(n_units)
    T = n_units + WINDOW + CHUNK + 8
    sign = torch.from_numpy(rng.choice([-1.0, 1.0], 128))
    val = span_values(kind, n_units, rng)
    rows = torch.from_numpy(val)[:, None] * sign[None, :]
    one_each = lambda n: [np.arange(n + 1)]
    for k_max, budget in ((7, 0), (0, n_units // 3 + 1), (n_units // 2 + 1, n_units // 4 + 2), (0, T)):
        w = Workload("mini-units", 4, 1, 128, "bf16", T, CHUNK, SINK, WINDOW, k_max, budget, "uniform", 16, 128)
        ctx = LtriContext(config_from_workload(w, n_layers=1, max_tokens=T, theta=1e30, max_spans=T, unit_tokens=1), gpu_device)
        ka, va = ctx.arena_views()
        ka.zero_(), va.zero_()
        ka[0, 0, 0, :n_units].copy_(rows.to(torch.bfloat16))
        for n in (1, CHUNK):
            ctx.reset(0)
            for at in range(0, n_units, CHUNK):
                m = min(CHUNK, n_units - at)
                ctx.append_chunk_with_spans(0, 0, m, one_each(m))
            ctx.append_chunk_with_spans(0, 0, WINDOW, one_each(WINDOW))
            ctx.append_chunk_with_spans(0, 0, n, one_each(n))
            q = sign.to(torch.bfloat16).to(gpu_device).expand(1, n, 4, 128).contiguous()
            ctx.retrieve(0, 0, 1, q)
            clip = (np.arange(n_units) >= SINK).astype(int)
            want = select_reference(val, clip, k_max, budget)
            ids, _ = ctx.get_selection(0, 0, 0)
            assert list(ids) == want, (k_max, budget, n)
            here = n_units + WINDOW
            assert list(ctx.get_token_list(0, 0, 0)) == list(range(SINK)) + want + list(range(here - WINDOW, here))
        assert ctx.sync_status() == 0
