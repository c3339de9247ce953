"""Step 2 of a chunk: how many sequences a trip of launches takes, against the room of the buffer that the pieces and running
sums of its query rows lie in; and step 2 of many sequences with index vectors on either side of the longest table that the
one-launch kernel takes."""
import ctypes as C
import shutil
import subprocess

import pytest
import torch

import __graft_entry__ as build_entry
from paper_2412_04757_amd import LtriContext, config_from_workload
from workloads import Workload, theta_default

PROGRAM = r"""
#include <stdio.h>
#include "retrieve_shape.h"
int main() {
  int sums, votes, stored, n_q, bytes, spans, items, count, heads, room;
  while (scanf("%d %d %d %d %d %d %d %d %d %d", &sums, &votes, &stored, &n_q, &bytes, &spans, &items, &count, &heads, &room) == 10) {
    const ltri::RetrieveShape s = ltri::retrieve_shape(sums, votes, stored, n_q, bytes, spans, items, count, heads, room);
    printf("%d %d %d %d %d %d %d %d\n", s.one_tail, s.from_sums, s.from_rows, s.spans, s.pieces, s.per, ltri::qrep_units(n_q),
           ltri::retrieve_reads_stored(n_q, bytes, spans, items, count, heads));
  }
}
"""
LONGEST = 5120          # spans: the longest table whose keys, ids and lengths fit the LDS beside the list's scratch


def test_pieces_and_running_sums_stay_inside_their_buffer(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    (tmp_path / "a.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-I" + build_entry.CSRC, str(tmp_path / "a.cpp"), "-o", str(tmp_path / "a")], check=True)
    calls = []
    for count in range(1, 65):
        for spans in (1, 130, LONGEST, LONGEST + 1, 8192, 8193, 60000):
            for n_q in (2, 128, 129, 1000, 2048):
                for sums, votes, stored, items in ((0, 0, 0, spans), (0, 0, 1, spans), (1, 0, 0, spans), (0, 1, 0, 100), (0, 0, 1, 100),
                                                   (0, 0, 1, 8192)):
                    bytes_ = (256, 2048, 4096)[(count + n_q) % 3]
                    calls.append((sums and n_q > 128, votes, stored, n_q, bytes_, spans, items, count, 2, min(count, 4)))
    text = "\n".join(" ".join(str(int(v)) for v in x) for x in calls)
    lines = subprocess.run([str(tmp_path / "a")], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(lines) == len(calls)
    for (sums, votes, stored, n_q, bytes_, spans, items, count, heads, room), line in zip(calls, lines):
        one, from_sums, from_rows, spans_, pieces, per, units, reads_stored = (int(v) for v in line.split())
        case = (sums, votes, stored, n_q, bytes_, spans, items, count)
        assert one == (not votes and spans <= 8192 and items <= LONGEST), case
        # what step 1 takes along is read by step 2, and not taken by it again
        assert reads_stored == (spans <= 8192 and items <= LONGEST and (n_q > 128 or n_q * bytes_ > 256 << 10 and count <= 4)), case
        if stored:
            assert reads_stored == (not from_rows and not spans_ and not pieces), case
        # Q^R has one source
        assert per >= 1 and from_sums + from_rows + spans_ + pieces == (not (stored and reads_stored)), case
        # buffer: two times `room` sequences' (Lp / 128 + Lp) rows, Lp the chunk rounded up to 64
        Lp = -(-n_q // 64) * 64
        for off in range(0, count, per):
            in_launch = min(per, count - off)
            if pieces:
                assert in_launch * units <= 2 * room * (Lp // 128 + Lp), case
            if pieces or from_sums:
                assert in_launch <= room, case


def guarded(ctx):
    """The context again, its scratch followed by a region that nothing may touch; the region."""
    guard = 1 << 20
    whole = torch.empty(ctx.scratch_bytes + guard, dtype=torch.uint8, device=ctx.device)
    whole.fill_(0xA5)
    assert ctx.lib.ltri_destroy(ctx.handle) == 0
    ctx.handle, ctx.scratch = C.c_void_p(), whole
    assert ctx.lib.ltri_create(C.byref(ctx.cfg), ctx.k_arena.data_ptr(), ctx.v_arena.data_ptr(), ctx.state.data_ptr(),
                               whole.data_ptr(), ctx.stream.cuda_stream, C.byref(ctx.handle)) == 0
    return whole[ctx.scratch_bytes:]


@pytest.mark.gpu
@pytest.mark.parametrize("kv_offload", [0, 1])
def test_step_of_many_sequences_with_a_long_table(gpu_device, kv_offload):
    """18 sequences with index vectors, whose tables may hold more spans than the one-launch kernel takes from chunk 21 on: one
    call per chunk and three calls select the same, and nothing behind the scratch buffer is written."""
    S, n, chunks = 18, 256, 23
    assert 20 * n <= LONGEST < (chunks - 1) * n
    w = Workload("mini-long", 2, 1, 128, "bf16", n * chunks, n, 4, 100, 0, 500, "uniform", 16, 200)
    gen = torch.Generator(device=gpu_device).manual_seed(3)
    T = n * chunks
    mean = torch.randn(S, 1, T // 50 + 1, 128, generator=gen, device=gpu_device).repeat_interleave(50, 2)[:, :, :T]
    K = (0.5 * (mean + 0.3 * torch.randn(S, 1, T, 128, generator=gen, device=gpu_device))).bfloat16()
    V = torch.randn(S, 1, T, 128, generator=gen, device=gpu_device).bfloat16()
    Q = torch.randn(S, T, 2, 128, generator=gen, device=gpu_device).bfloat16()
    got = []
    for step in (True, False):
        ctx = LtriContext(config_from_workload(w, n_layers=1, n_seqs=S, max_tokens=T, theta=theta_default(128) / 4, max_spans=T,
                                               rep_mode=1, lam=1.5, kv_offload=kv_offload), gpu_device)
        guard = guarded(ctx)
        res = []
        for at in range(0, T, n):
            k, v = K[:, :, at:at + n].contiguous(), V[:, :, at:at + n].contiguous()
            q = Q[:, at:at + n].contiguous()
            if step:
                out = ctx.step(0, 0, S, k, v, q)
            else:
                ctx.append_chunk(0, 0, S, n, k_chunk=k, v_chunk=v)
                ctx.retrieve(0, 0, S, q)
                out = ctx.attend(0, 0, S, q)
            if at >= T - 4 * n or at == 0:
                res.append((out, [(list(i), list(x)) for i, x in (ctx.get_selection(0, s, 0) for s in range(S))],
                            [list(ctx.get_token_list(0, s, 0)) for s in range(S)]))
        assert ctx.sync_status() == 0
        assert bool((guard == 0xA5).all())
        got.append(res)
    for (oa, sa, la), (ob, sb, lb) in zip(*got):
        assert sa == sb and la == lb
        # (the offloaded step rounds the first part's output once more: 2^-8 of it and of the result)
        assert torch.equal(oa, ob) if not kv_offload else float((oa - ob).norm() / ob.norm()) <= 2.0 ** -7


@pytest.mark.gpu
@pytest.mark.parametrize("rows,dtype,dim,kw", [
    (100, "bf16", 128, {}), (128, "bf16", 128, dict(rep_mode=1, lam=1.5)),                  # 16 heads: rows summed on the way, or before
    (200, "bf16", 128, dict(rep_mode=1, lam=1.5)), (300, "bf16", 128, dict(rep_mode=1, lam=1.5, unit_tokens=64)), (129, "f32", 64, {}),
])
def test_sequences_together_and_alone(gpu_device, rows, dtype, dim, kw):
    """Q^R comes from different launches for 18 sequences and for one, and several trips of sums share one selection: the selections
    are the same (sums of bf16 values are exact; fp32 ones in fp64 differ by less than the scores do)."""
    S, hist = 18, 900
    w = Workload("mini-together", 16, 1, dim, dtype, hist + rows, 300, 4, 60, 0, 300, "uniform", 16, 200)
    ctx = LtriContext(config_from_workload(w, n_layers=1, n_seqs=S, max_tokens=hist + rows, max_spans=hist + rows,
                                           theta=theta_default(dim) / 4, **kw), gpu_device)
    gen = torch.Generator(device=gpu_device).manual_seed(rows)
    ka, va = ctx.arena_views()
    T = hist + rows
    mean = torch.randn(S, 1, T // 30 + 1, dim, generator=gen, device=gpu_device).repeat_interleave(30, 2)[:, :, :T]
    ka[0].copy_(0.5 * (mean + 0.3 * torch.randn(S, 1, T, dim, generator=gen, device=gpu_device)))
    va.copy_(torch.randn(va.shape, generator=gen, device=gpu_device))
    for c0 in range(0, hist, 300):
        ctx.append_chunk(0, 0, S, 300)
    ctx.append_chunk(0, 0, S, rows)
    q = torch.randn(S, rows, 16, dim, generator=gen, device=gpu_device).to(ka.dtype)
    lists = lambda s: (list(ctx.get_selection(0, s, 0)[0]), list(ctx.get_token_list(0, s, 0)))
    ctx.retrieve(0, 0, S, q)
    together = [lists(s) for s in range(S)]
    for s in range(S):
        ctx.retrieve(0, s, 1, q[s:s + 1].contiguous())
        assert lists(s) == together[s], s
    assert ctx.sync_status() == 0
    assert len({tuple(t[0]) for t in together}) > S // 2
