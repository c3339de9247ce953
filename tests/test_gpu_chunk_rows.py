"""Rows that come with a call against rows that are in the arenas already, at chunk lengths around the tile, the sizes where
the merge of the tiles' results moves into the selection, and the copy's whole workgroups."""
import pytest
import torch

from paper_2412_04757_amd import LtriContext, config_from_workload
from tests.test_gpu_parity import _stream_parity
from workloads import Workload, theta_default

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[256, 257, 64, 65], [1024, 1025], [1025, 960, 961]])
def test_merge_of_tiles_at_its_limits(gpu_device, sizes):
    w = Workload("mini-merge", 4, 1, 128, "bf16", sum(sizes), max(sizes), 4, 96, 0, 300, "uniform", 16, 200)
    _stream_parity(w, 31, sum(sizes), gpu_device, chunk_sizes=sizes, whole_step=True)


@pytest.mark.parametrize("whole_step", [True, False])
@pytest.mark.parametrize("dtype,dim,seqs", [("bf16", 128, 1), ("bf16", 128, 5), ("f32", 64, 2)])
def test_rows_passed_equal_rows_in_place(gpu_device, dtype, dim, seqs, whole_step):
    sizes = [2, 65, 256, 700, 1, 3, 1025, 1]
    T = sum(sizes)
    w = Workload("mini-rows", 4, 2, dim, dtype, T, max(sizes), 4, 100, 0, 300, "uniform", 16, 200)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=gpu_device).manual_seed(5)
    mean = torch.randn(seqs, 2, T // 50 + 1, dim, generator=gen, device=gpu_device).repeat_interleave(50, 2)[:, :, :T]
    K = (mean + 0.3 * torch.randn(seqs, 2, T, dim, generator=gen, device=gpu_device)).to(dt)
    V = torch.randn(seqs, 2, T, dim, generator=gen, device=gpu_device).to(dt)
    Q = torch.randn(seqs, T, 4, dim, generator=gen, device=gpu_device).to(dt)
    got = []
    for passed in (True, False):
        ctx = LtriContext(config_from_workload(w, n_layers=1, n_seqs=seqs, max_tokens=T, theta=theta_default(dim)), gpu_device)
        ka, va = ctx.arena_views()
        ka.zero_(), va.zero_()
        outs, at = [], 0
        for n in sizes:
            k, v = K[:, :, at:at + n].contiguous(), V[:, :, at:at + n].contiguous()
            if not passed:
                ka[0, :, :, at:at + n].copy_(k), va[0, :, :, at:at + n].copy_(v)
                k = v = None
            q = Q[:, at:at + n].contiguous()
            if whole_step:
                outs.append(ctx.step(0, 0, seqs, k, v, q))
            else:
                ctx.append_chunk(0, 0, seqs, n, k_chunk=k, v_chunk=v)
                ctx.retrieve(0, 0, seqs, q)
                outs.append(ctx.attend(0, 0, seqs, q))
            at += n
        assert ctx.sync_status() == 0
        spans = [[list(x) for x in ctx.get_spans(0, s, h)] + [ctx.get_rep_keys(0, s, h)] for s in range(seqs) for h in range(2)]
        got.append((outs, spans, ka.clone(), va.clone()))
    (oa, sa, ka, va), (ob, sb, kb, vb) = got
    assert torch.equal(ka, kb) and torch.equal(va, vb) and torch.equal(ka[0, :, :, :T], K)
    for a, b in zip(sa, sb):
        assert a[:2] == b[:2] and torch.equal(a[2], b[2])
    for a, b in zip(oa, ob):
        assert torch.equal(a, b)


@pytest.mark.parametrize("kw", [dict(), dict(rep_mode=1, lam=1.5, unit_tokens=128, index_block_max=12), dict(rep_mode=1, lam=1.5)])
@pytest.mark.parametrize("seqs", [1, 6])
def test_step_equals_calls(gpu_device, seqs, kw):
    """Several batches of sequences (six, four to a segmentation launch) and index vectors: in one call, where steps 1 and 2 of a
    batch follow each other and Q^R comes from step 1's launches, and in three. Sums of bf16 values are exact, so all is equal."""
    sizes = [300, 129, 2048, 200]
    T = sum(sizes)
    w = Workload("mini-calls", 8, 2, 128, "bf16", T, max(sizes), 4, 100, 0, 500, "uniform", 16, 200)
    gen = torch.Generator(device=gpu_device).manual_seed(9)
    mean = torch.randn(seqs, 2, T // 50 + 1, 128, generator=gen, device=gpu_device).repeat_interleave(50, 2)[:, :, :T]
    K = 0.5 * (mean + 0.3 * torch.randn(seqs, 2, T, 128, generator=gen, device=gpu_device))
    V = torch.randn(seqs, 2, T, 128, generator=gen, device=gpu_device)
    Q = torch.randn(seqs, T, 8, 128, generator=gen, device=gpu_device).bfloat16()
    got = []
    for step in (True, False):
        ctx = LtriContext(config_from_workload(w, n_layers=1, n_seqs=seqs, max_tokens=T, theta=theta_default(128) / 4, **kw), gpu_device)
        ka, va = ctx.arena_views()
        ka[0].copy_(K), va[0].copy_(V)
        res, at = [], 0
        for n in sizes:
            q = Q[:, at:at + n].contiguous()
            if step:
                out = ctx.step(0, 0, seqs, None, None, q)
            else:
                ctx.append_chunk(0, 0, seqs, n)
                ctx.retrieve(0, 0, seqs, q)
                out = ctx.attend(0, 0, seqs, q)
            sel = [ctx.get_selection(0, s, h) for s in range(seqs) for h in range(2)]
            res.append((out, [(list(i), list(x)) for i, x in sel], [list(ctx.get_token_list(0, s, h)) for s in range(seqs) for h in range(2)]))
            at += n
        assert ctx.sync_status() == 0
        got.append(res)
    for (oa, sa, la), (ob, sb, lb) in zip(*got):
        assert sa == sb and la == lb and torch.equal(oa, ob)


@pytest.mark.parametrize("seqs,rows", [(3, 3), (12, 3), (33, 2), (40, 4), (12, 100)])
def test_retrieve_of_many_sequences(gpu_device, seqs, rows):
    """The scoring workgroups of a sequence and KV head become fewer as there are more of those (24, 96, 264, 320): the
    selections of a call for all sequences are those of a call for each."""
    spans = 400 + 16 * torch.arange(seqs) % 300          # stored spans of a sequence, 3 tokens each
    T = 3 * 700 + 40 + rows
    w = Workload("mini-many", 8, 8, 128, "bf16", T, 256, 4, 40, 0, 300, "uniform", 16, 200)
    ctx = LtriContext(config_from_workload(w, n_layers=1, n_seqs=seqs, max_tokens=T, theta=1e30, max_spans=1024), gpu_device)
    gen = torch.Generator(device=gpu_device).manual_seed(seqs)
    for a in ctx.arena_views():
        a.copy_(torch.randn(a.shape, generator=gen, device=gpu_device))
    for s in range(seqs):
        for at in range(0, int(spans[s]), 80):
            n = min(80, int(spans[s]) - at)
            ctx.append_chunk_with_spans(0, s, 3 * n, [list(range(0, 3 * n + 1, 3))] * 8)
        ctx.append_chunk_with_spans(0, s, 40, [[0, 40]] * 8)
    ctx.append_chunk(0, 0, seqs, rows)
    q = torch.randn(seqs, rows, 8, 128, generator=gen, device=gpu_device).bfloat16()
    lists = lambda s: [(list(ctx.get_selection(0, s, h)[0]), list(ctx.get_token_list(0, s, h))) for h in range(8)]
    ctx.retrieve(0, 0, seqs, q)
    together = [lists(s) for s in range(seqs)]
    for s in range(seqs):
        ctx.retrieve(0, s, 1, q[s:s + 1].contiguous())
        assert lists(s) == together[s], s
    assert ctx.sync_status() == 0
    assert len({tuple(l[0]) for t in together for l in t}) > seqs
