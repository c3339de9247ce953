"""The shapes the matrix-core attention chooses by the size of a launch (one or two key groups per workgroup, a key
range split over workgroups with partial results merged afterwards): every row and head against an fp64 reference on
the device's own token lists, at row counts and context lengths around the edges of tiles, stages and sub-tiles."""
import math

import pytest
import torch

from paper_2412_04757_amd import LtriContext, config_from_workload
from workloads import Workload, planted_stream, theta_default

pytestmark = pytest.mark.gpu


def attend_reference(ctx, w, seq, c0, q):
    """fp64 attention of q [n][Hq][d] over the context list and the chunk that starts at c0; output and log-sum-exp."""
    ka, va = ctx.arena_views()
    n, G = q.shape[0], w.n_q_heads // w.n_kv_heads
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    lse = torch.empty(q.shape[:2], dtype=torch.float64, device=q.device)
    for h in range(w.n_kv_heads):
        t = torch.from_numpy(ctx.get_token_list(0, seq, h)).long().to(q.device)
        rows = torch.cat([t, torch.arange(c0, c0 + n, device=q.device)])
        K, V = ka[0, seq, h, rows].double(), va[0, seq, h, rows].double()
        future = torch.arange(len(rows), device=q.device)[None, :] > len(t) + torch.arange(n, device=q.device)[:, None]
        for g in range(h * G, (h + 1) * G):
            z = (q[:, g].double() @ K.t().contiguous()) / math.sqrt(w.head_dim)
            z.masked_fill_(future, -math.inf)
            out[:, g] = torch.softmax(z, 1) @ V
            lse[:, g] = torch.logsumexp(z, 1)
    return out, lse


# (query heads, KV heads, sequences, window, budget, history, query rows)
SHAPES = [
    (8, 2, 1, 64, 0, 0, 5),            # no context at all: a lone chunk tile, splits would be empty
    (8, 2, 1, 60, 64, 700, 33),        # a list of whole tiles (4 + 64 + 60), a second sub-tile of one row
    (8, 2, 1, 123, 100, 900, 64),      # an odd number of tiles, a ragged last context tile
    (32, 8, 1, 1024, 1024, 4096, 128),  # two groups and several splits
    (32, 8, 1, 900, 700, 4096, 301),
    (32, 8, 4, 200, 300, 1500, 256),   # a batch, two groups without a split
    (32, 8, 1, 1024, 2048, 6000, 1199),
    (8, 8, 3, 130, 200, 1000, 97),     # one query head per KV head: four (two groups) or eight row sub-tiles
    (16, 8, 1, 333, 444, 2000, 130),   # two
    (24, 2, 1, 500, 0, 1000, 70),      # three workgroups per KV head, everything retrieved
]


@pytest.mark.parametrize("hq,hkv,seqs,window,budget,history,rows", SHAPES)
def test_attention_launch_shapes(gpu_device, hq, hkv, seqs, window, budget, history, rows):
    w = Workload("shapes", hq, hkv, 128, "bf16", history + rows, 2048, 4, window, 0, budget, "uniform", 16, 96)
    cfg = config_from_workload(w, theta=theta_default(128), n_layers=1, n_seqs=seqs)
    ctx = LtriContext(cfg, gpu_device)
    ka, va = ctx.arena_views()
    q = []
    for s in range(seqs):
        K, V, Q, _ = planted_stream(w, 900 + s, device=str(gpu_device), context=history + rows)
        ka[0, s].copy_(K)
        va[0, s].copy_(V)
        q.append(Q[history:])
    for c0 in range(0, history, 512):
        ctx.append_chunk(0, 0, seqs, min(512, history - c0))
    q = torch.stack(q).contiguous()
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device=gpu_device)
    out = torch.full_like(q, float("nan"))
    ctx.append_chunk(0, 0, seqs, rows)
    ctx.retrieve(0, 0, seqs, q)
    ctx.attend(0, 0, seqs, q, out=out, lse=lse)
    again = torch.full_like(q, float("nan"))
    ctx.attend_static(0, 0, seqs, q, again)           # the same launch (the buffer of short blocks is not used)
    assert torch.equal(out, again)
    for s in range(seqs):
        want, want_lse = attend_reference(ctx, w, s, history, q[s])
        # probabilities and output rounded to bf16 (2^-9 each of values below a few units), fp32 sums
        assert float((out[s].double() - want).abs().max()) <= 2e-2
        assert float((lse[s].double() - want_lse).abs().max()) <= 2e-3
    assert ctx.sync_status() == 0


def test_attention_scores_that_keep_growing(gpu_device):
    """Scores whose running maximum climbs through the whole context by far more than the slack of the rescale: keys of
    later tokens are longer, so that nearly all weight sits on the last keys and every tile moves the reference."""
    w = Workload("growing", 8, 2, 128, "bf16", 2048 + 64, 512, 4, 2048, 0, 64, "uniform", 16, 96)
    cfg = config_from_workload(w, theta=theta_default(128), n_layers=1, n_seqs=1)
    ctx = LtriContext(cfg, gpu_device)
    ka, va = ctx.arena_views()
    g = torch.Generator(device=str(gpu_device)).manual_seed(5)
    base = torch.randn((2, 1, 128), generator=g, device=gpu_device)
    grow = torch.linspace(0.0, 6.0, 2048 + 64, device=gpu_device)[None, :, None]
    ka[0, 0].copy_(base * grow)
    va[0, 0].copy_(torch.randn(va[0, 0].shape, generator=g, device=gpu_device))
    q = (base.repeat_interleave(4, 0)[:, 0] + 0.1 * torch.randn((64, 8, 128), generator=g, device=gpu_device)).bfloat16()
    for c0 in range(0, 2048, 512):
        ctx.append_chunk(0, 0, 1, 512)
    ctx.append_chunk(0, 0, 1, 64)
    ctx.retrieve(0, 0, 1, q.unsqueeze(0).contiguous())
    lse = torch.empty((1, 64, 8), dtype=torch.float32, device=gpu_device)
    out = ctx.attend(0, 0, 1, q.unsqueeze(0).contiguous(), lse=lse)
    want, want_lse = attend_reference(ctx, w, 0, 2048, q)
    assert float((out[0].double() - want).abs().max()) <= 2e-2
    assert float((lse[0].double() - want_lse).abs().max()) <= 2e-3
