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


def worst_row(got, want):
    """Largest error of a row (one query and head) relative to the row: 2-norms over head_dim."""
    return float(((got.double() - want).norm(dim=-1) / want.norm(dim=-1)).max())


# Bound of worst_row in bf16: the output is rounded to 2^-8 of itself, and so is every probability; over values that are
# random and zero in the mean, as here, the second adds up to no more than the first (both are sums of w_i v_i, one of
# them with factors below 2^-8). A key among 3000 is 1 / sqrt(3000) = 1.8e-2 of its row.
BF16_ROW = 2.0 ** -7

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
        assert worst_row(out[s], want) <= BF16_ROW
        # the log-sum-exp is that of the rounded probabilities: 2^-8 at the very most
        assert float((lse[s].double() - want_lse).abs().max()) <= 2e-3
    assert ctx.sync_status() == 0


def test_attention_scores_that_keep_growing(gpu_device):
    """Scores whose running maximum climbs through the whole context: keys of later tokens are longer, so that nearly all
    weight sits on the last keys and every tile moves the reference."""
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
    assert worst_row(out[0], want) <= BF16_ROW
    assert float((lse[0].double() - want_lse).abs().max()) <= 2e-3


@pytest.mark.parametrize("hq,hkv,seqs,window,budget,history,rows",
                         SHAPES + [(32, 8, 1, 1000, 500, 1800, 2048), (8, 2, 1, 1000, 500, 1800, 3)])
def test_every_key_counts_once(gpu_device, hq, hkv, seqs, window, budget, history, rows):
    """All keys are zero, so every visible key has the same weight, exactly, and every value is 1 in one of the 128 columns
    and 0 elsewhere: an output times the number of keys is a count of at most a hundred keys or so, which bf16 holds, and
    the log-sum-exp is the logarithm of the number. A key lost, added or counted twice at an edge of a tile, stage, split or
    sub-tile shows in every row that it belongs to."""
    w = Workload("count", hq, hkv, 128, "bf16", history + rows, 2048, 4, window, 0, budget, "uniform", 16, 96)
    ctx = LtriContext(config_from_workload(w, theta=theta_default(128), n_layers=1, n_seqs=seqs), gpu_device)
    ka, va = ctx.arena_views()
    gen = torch.Generator(device=gpu_device).manual_seed(21)
    column = torch.randint(0, 128, va.shape[:-1], generator=gen, device=gpu_device)
    ka.zero_()
    va.zero_()
    va.scatter_(-1, column.unsqueeze(-1), 1.0)
    for c0 in range(0, history, 450):
        ctx.append_chunk(0, 0, seqs, min(450, history - c0))
    ctx.append_chunk(0, 0, seqs, rows)
    q = torch.randn((seqs, rows, hq, 128), generator=gen, device=gpu_device).to(torch.bfloat16)
    ctx.retrieve(0, 0, seqs, q)
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device=gpu_device)
    out = ctx.attend(0, 0, seqs, q, lse=lse).double()
    G = hq // hkv
    for s in range(seqs):
        for h in range(hkv):
            t = torch.from_numpy(ctx.get_token_list(0, s, h)).long().to(gpu_device)
            one = torch.nn.functional.one_hot(column[0, s, h], 128).double()
            count = one[t].sum(0) + one[history:history + rows].cumsum(0)             # [rows][128]
            n = count.sum(1)
            assert float(count.max()) < 120                 # one key more or less is over 2^-7 of a column
            got = out[s, :, h * G:(h + 1) * G] * n[:, None, None]
            assert bool(((got - count[:, None]).abs() <= 2.0 ** -8 * count[:, None]).all())
            assert float((lse[s, :, h * G:(h + 1) * G].double() - n.log()[:, None]).abs().max()) <= 2e-6
    assert ctx.sync_status() == 0


def test_step_timing_covers_the_merge(gpu_device):
    """Steps whose attention is split: a record each, from the start of the attention to the end of the merge behind it."""
    w = Workload("timing", 32, 8, 128, "bf16", 8192, 1024, 4, 1024, 0, 1024, "uniform", 16, 96)
    ctx = LtriContext(config_from_workload(w, theta=theta_default(128), n_layers=1, n_seqs=1), gpu_device)
    K, V, Q, _ = planted_stream(w, 3, device=str(gpu_device), context=8192)
    ka, va = ctx.arena_views()
    ka[0, 0], va[0, 0] = K, V
    ctx.set_step_timing(True)
    sizes, at = [1024] * 4 + [128] * 8, 0
    for n in sizes:
        ctx.step(0, 0, 1, None, None, Q[at:at + n].contiguous())
        at += n
    ms, rest = ctx.read_step_timing()
    assert len(ms) == len(sizes) and not rest.any()
    # between a launch over one tile and a millisecond, which is ten times what any of them takes
    assert bool((ms > 2e-3).all()) and bool((ms[1:] < 1.0).all()), ms


def test_rounding_of_a_batch(gpu_device):
    """A launch is shaped by all of its sequences, so the same chunk rounds differently alone, in a batch and beside a longer
    neighbour; each time it is within the rounding of bf16 of the exact result, and the same tokens are attended."""
    lens = [900, 900, 4100]
    rows, hq, hkv = 150, 32, 8
    w = Workload("batch", hq, hkv, 128, "bf16", max(lens) + rows, 2048, 4, 300, 0, 400, "uniform", 16, 96)
    cfg = config_from_workload(w, theta=theta_default(128), n_layers=1, n_seqs=3)
    K, V, Q, _ = planted_stream(w, 77, device=str(gpu_device), context=max(lens) + rows)
    q1 = Q[900:900 + rows]
    outs = []
    for batch in (1, 2, 3):                    # alone, with an equal sequence, with a longer one as well
        ctx = LtriContext(cfg, gpu_device)
        ka, va = ctx.arena_views()
        ka[0], va[0] = K, V
        for s in range(3):
            for c0 in range(0, lens[s], 900):
                ctx.append_chunk(0, s, 1, min(900, lens[s] - c0))
        q = q1.expand(batch, rows, hq, 128).contiguous()
        ctx.append_chunk(0, 0, batch, rows)
        ctx.retrieve(0, 0, batch, q)
        out = ctx.attend(0, 0, batch, q)
        want, _ = attend_reference(ctx, w, 0, 900, q1)
        assert worst_row(out[0], want) <= BF16_ROW
        outs.append((out[0].double(), [list(ctx.get_token_list(0, 0, h)) for h in range(hkv)]))
        assert ctx.sync_status() == 0
    for out, lists in outs[1:]:
        assert lists == outs[0][1]
        assert worst_row(out, outs[0][0]) <= BF16_ROW


@pytest.mark.parametrize("hq,hkv,seqs,window,history,rows", [
    (32, 8, 1, 1000, 1500, 2048),      # a full chip: every wavefront on all keys
    (32, 8, 1, 1000, 1500, 1024),      # two key groups
    (8, 2, 1, 1000, 1500, 65),         # two key groups and splits
    (8, 2, 1, 1000, 1500, 3),
])
def test_keys_that_raise_the_maximum_count_exactly(gpu_device, hq, hkv, seqs, window, history, rows):
    """A key per context tile scores a little more than the one before, all others nothing. The probability of each is
    taken when it is the maximum, where it is 1 and needs no rounding; what is left of it later is an fp32 factor. So the
    output, in which the values of those keys nearly cancel, is off by its own rounding and fp32 sums only."""
    w = Workload("records", hq, hkv, 128, "bf16", history + rows, 2048, 4, window, 0, 16, "uniform", 16, 96)
    ctx = LtriContext(config_from_workload(w, theta=theta_default(128), n_layers=1, n_seqs=seqs), gpu_device)
    ka, va = ctx.arena_views()
    gen = torch.Generator(device=gpu_device).manual_seed(11)
    ka.zero_()
    ka[..., 0] = -4096.0
    va.copy_(torch.randint(0, 2, va.shape, generator=gen, device=gpu_device) * 2 - 1)
    # list entries 20 (or 4 fewer, as many tokens as are retrieved): the window's tokens from w0 on; one key per 64 of them
    at = torch.arange(history - window + 30, history, 64, device=gpu_device)
    ka[..., at, 0] = (8.0 + 0.125 * torch.arange(len(at), device=gpu_device)).to(torch.bfloat16)
    q = torch.zeros((seqs, rows, hq, 128), dtype=torch.bfloat16, device=gpu_device)
    q[..., 0] = 1.0 + 2.0 * torch.rand((seqs, rows, hq), generator=gen, device=gpu_device)
    for c0 in range(0, history, 750):
        ctx.append_chunk(0, 0, seqs, min(750, history - c0))
    ctx.append_chunk(0, 0, seqs, rows)
    ctx.retrieve(0, 0, seqs, q)
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device=gpu_device)
    out = ctx.attend(0, 0, seqs, q, lse=lse)
    for s in range(seqs):
        want, want_lse = attend_reference(ctx, w, s, history, q[s])
        # bf16 output: 2^-8 of itself; fp32: scores up to 8 (2^-24 each of a product and a sum), 16 keys, sums up to 16
        assert bool(((out[s].double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all())
        assert float((lse[s].double() - want_lse).abs().max()) <= 1e-5
    assert ctx.sync_status() == 0


# fp32: (query heads, KV heads, head_dim, sequences, window, budget, history, query rows)
F32_SHAPES = [
    (4, 1, 64, 1, 64, 0, 0, 2),          # fewer tiles than wavefronts, no context
    (4, 1, 64, 1, 11, 0, 40, 1),         # one row; a context of one ragged tile
    (4, 1, 64, 1, 512, 512, 1500, 256),
    (6, 2, 64, 2, 100, 77, 700, 85),     # a group of three heads: the last workgroup's pairs are ragged
    (1, 1, 128, 1, 60, 64, 700, 33),     # one head: 16 rows per workgroup
    (40, 2, 128, 1, 123, 100, 900, 7),   # more heads than pairs of a workgroup
    (4, 2, 128, 3, 130, 200, 1000, 97),
]


@pytest.mark.parametrize("hq,hkv,dim,seqs,window,budget,history,rows", F32_SHAPES)
def test_fp32_attention(gpu_device, hq, hkv, dim, seqs, window, budget, history, rows):
    """Every row and head against the fp64 reference; then with an infinity in the values of the chunk's last token,
    which only the last row sees."""
    w = Workload("f32", hq, hkv, dim, "f32", history + rows, 256, 4, window, 0, budget, "uniform", 8, 48)
    ctx = LtriContext(config_from_workload(w, theta=theta_default(dim), n_layers=1, n_seqs=seqs), gpu_device)
    ka, va = ctx.arena_views()
    q = []
    for s in range(seqs):
        K, V, Q, _ = planted_stream(w, 700 + s, device=str(gpu_device), context=history + rows)
        ka[0, s].copy_(K)
        va[0, s].copy_(V)
        q.append(Q[history:])
    for c0 in range(0, history, 256):
        ctx.append_chunk(0, 0, seqs, min(256, history - c0))
    q = torch.stack(q).contiguous()
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device=gpu_device)
    out = torch.full_like(q, float("nan"))
    ctx.append_chunk(0, 0, seqs, rows)
    ctx.retrieve(0, 0, seqs, q)
    ctx.attend(0, 0, seqs, q, out=out, lse=lse)
    for s in range(seqs):
        want, want_lse = attend_reference(ctx, w, s, history, q[s])
        # scores of up to 128 fp32 products of values around 1 and |score| <= 8: 128 * 2^-24 * 8 at the very most in the
        # exponent, as a relative error of the weights; the sums of weights and outputs (below a few units) add less
        assert float((out[s].double() - want).abs().max()) <= 6e-5
        assert float((lse[s].double() - want_lse).abs().max()) <= 6e-5
    va[0, :, :, history + rows - 1] = float("inf")
    poisoned = torch.full_like(q, float("nan"))
    ctx.attend(0, 0, seqs, q, out=poisoned)
    # the last tile's 16 keys are then added one by one: 16 roundings of sums below 4 (2^-23 each) in another order
    assert bool(((poisoned[:, :-1] - out[:, :-1]).abs() <= 4e-6).all())
    assert not torch.isfinite(poisoned[:, -1]).any()
    assert ctx.sync_status() == 0
