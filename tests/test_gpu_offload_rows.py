"""Host-offloaded keys and values: the host arenas after ltri_step, whose rows go out with the fetch of the retrieved
ones, and after the three calls, whose rows the append writes."""
import pytest
import torch

from paper_2412_04757_amd import LtriContext, config_from_workload
from workloads import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entry", ["step", "calls"])
@pytest.mark.parametrize("sizes", [[1, 5, 300, 129, 64], [512, 512, 4, 77]])
def test_host_arenas_hold_every_row(gpu_device, entry, sizes):
    T, S, Hq, H, d = 1200, 2, 8, 2, 128
    w = Workload("mini-rows", Hq, H, d, "bf16", T, 512, 4, 96, 0, 200, "uniform", 16, 96)
    ctx = LtriContext(config_from_workload(w, n_layers=1, n_seqs=S, max_tokens=T, theta=5.0, max_spans=T, kv_offload=1), gpu_device)
    ka, va = ctx.arena_views()
    ka.fill_(-3.0), va.fill_(-3.0)
    gen = torch.Generator(device=gpu_device).manual_seed(3)
    draw = lambda *s: torch.randn(s, generator=gen, device=gpu_device).to(torch.bfloat16)
    K, V = draw(S, H, sum(sizes), d), draw(S, H, sum(sizes), d)
    at = 0
    for n in sizes:
        k, v, q = K[:, :, at:at + n].contiguous(), V[:, :, at:at + n].contiguous(), draw(S, n, Hq, d)
        if entry == "step":
            ctx.step(0, 0, S, k, v, q)
        else:
            ctx.append_chunk(0, 0, S, n, k_chunk=k, v_chunk=v)
            ctx.retrieve(0, 0, S, q)
            ctx.attend(0, 0, S, q)
        at += n
        assert ctx.sync_status() == 0
        assert torch.equal(ka[0, :, :, :at].cpu(), K[:, :, :at].cpu()) and torch.equal(va[0, :, :, :at].cpu(), V[:, :, :at].cpu())
        assert bool((ka[0, :, :, at:] == -3.0).all()) and bool((va[0, :, :, at:] == -3.0).all())
