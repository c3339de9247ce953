"""The scratch buffer holds temporaries of a call: between calls it may be overwritten, or lent to another context. Counters that
launches leave at zero for the next ones lie in the state buffer."""
import ctypes as C

import pytest
import torch

from paper_2412_04757_amd import LtriContext, config_from_workload
from workloads import Workload, theta_default

pytestmark = pytest.mark.gpu

# name: (query heads, KV heads, head_dim, dtype, sequences, window and budget), chunk lengths, further settings
CASES = {
    "decoding": ((8, 2, 128, "bf16", 3, 256), [600, 1, 1, 3, 1], {}),
    "short chunks by units": ((8, 2, 128, "bf16", 6, 256), [256, 100, 256, 7], dict(rep_mode=1, lam=1.5, unit_tokens=128, index_block_max=12)),
    "index vectors": ((8, 2, 128, "bf16", 2, 256), [700, 300, 130], dict(rep_mode=1, lam=1.5)),
    "even shares": ((32, 8, 128, "bf16", 1, 1024), [2048, 2048, 1050], {}),
    "fp32": ((4, 1, 64, "f32", 1, 256), [256, 256, 256, 256, 256, 1, 256], {}),
    "paper": ((8, 2, 128, "bf16", 1, 256), [128, 256, 128, 128], dict(seg_map=0, theta_quantile=0.9, phi=0.1, rep_mode=1, unit_tokens=128, max_spans=640)),
}


def stream(name, device, seed):
    (hq, hkv, dim, dtype, seqs, near), sizes, kw = CASES[name]
    T = sum(sizes)
    w = Workload("scratch", hq, hkv, dim, dtype, T, max(sizes), 4, near, 0, near, "uniform", 16, 200)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=device).manual_seed(seed)
    mean = torch.randn(seqs, hkv, T // 50 + 1, dim, generator=gen, device=device).repeat_interleave(50, 2)[:, :, :T]
    K = (mean + 0.3 * torch.randn(seqs, hkv, T, dim, generator=gen, device=device)).to(dt)
    V = torch.randn(seqs, hkv, T, dim, generator=gen, device=device).to(dt)
    Q = torch.randn(seqs, T, hq, dim, generator=gen, device=device).to(dt)
    ctx = LtriContext(config_from_workload(w, n_layers=1, n_seqs=seqs, max_tokens=T, theta=theta_default(dim), **kw), device)
    return ctx, seqs, sizes, K, V, Q


def lend(ctx, buffer):
    """The context again, on that scratch buffer."""
    assert buffer.numel() >= ctx.scratch_bytes and ctx.lib.ltri_destroy(ctx.handle) == 0
    ctx.handle, ctx.scratch = C.c_void_p(), buffer
    assert ctx.lib.ltri_create(C.byref(ctx.cfg), ctx.k_arena.data_ptr(), ctx.v_arena.data_ptr(), ctx.state.data_ptr(),
                               buffer.data_ptr(), ctx.stream.cuda_stream, C.byref(ctx.handle)) == 0


def calls(ctx, seqs, sizes, K, V, Q):
    """Every call of a stream in turn, by ltri_step and by the three calls; yields before each, and the outputs at the end."""
    outs, at = [], 0
    for i, n in enumerate(sizes):
        k, v, q = K[:, :, at:at + n].contiguous(), V[:, :, at:at + n].contiguous(), Q[:, at:at + n].contiguous()
        yield None
        if i % 2:
            outs.append(ctx.step(0, 0, seqs, k, v, q))
        else:
            ctx.append_chunk(0, 0, seqs, n, k_chunk=k, v_chunk=v)
            yield None
            ctx.retrieve(0, 0, seqs, q)
            yield None
            outs.append(ctx.attend(0, 0, seqs, q))
        at += n
    assert ctx.sync_status() == 0
    yield outs


def run(it, between=lambda: None):
    for x in it:
        if x is not None:
            return x
        between()


@pytest.mark.parametrize("name", CASES)
def test_scratch_may_be_overwritten_between_calls(gpu_device, name):
    want = run(calls(*stream(name, gpu_device, 1)))
    args = stream(name, gpu_device, 1)
    got = run(calls(*args), lambda: args[0].scratch.fill_(0xFF))
    for a, b in zip(want, got):
        assert torch.isfinite(a).all() and torch.equal(a, b)


def test_contexts_of_different_shapes_share_a_scratch(gpu_device):
    want = {name: run(calls(*stream(name, gpu_device, 2))) for name in CASES}
    args = {name: stream(name, gpu_device, 2) for name in CASES}
    buffer = torch.full((max(a[0].scratch_bytes for a in args.values()),), 0x7F, dtype=torch.uint8, device=gpu_device)
    for a in args.values():
        lend(a[0], buffer)
    live, got = {name: calls(*a) for name, a in args.items()}, {}
    while live:                                          # a call of each in turn
        for name in list(live):
            x = next(live[name])
            if x is not None:
                got[name] = x
                del live[name]
    for name in CASES:
        assert all(torch.equal(a, b) for a, b in zip(want[name], got[name])), name
