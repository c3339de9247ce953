"""The percentile threshold of step 1 at the chunk lengths where its selection changes method."""
import numpy as np
import pytest
import torch

from oracle import ltri_oracle as O
from paper_2412_04757_amd import LtriContext, config_from_workload
from paper_2412_04757_amd.binding import MAP_LOGIT, MAP_SOFTMAX
from workloads import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keys", ["normal", "constant", "halves"])
@pytest.mark.parametrize("chunk", [2, 3, 22, 23, 64, 65, 128, 180, 181, 200, 300])
def test_percentile_theta_around_the_list(gpu_device, chunk, keys):
    """Chunks whose cells are few enough to be ranked directly (22 tokens: 253), to be collected by the first pass
    (180 tokens: 16290), and just too many for that; random keys, and keys that tie all or most cells. The device's
    cells carry fp32 matrix-core error, so the values agree to 1e-5 of the map's largest cell, and on tied maps that
    tells a right digit from a wrong one."""
    w = Workload("mini-percentile", 8, 2, 128, "bf16", 1024, 512, 4, 128, 0, 300, "uniform", 16, 128)
    gen = torch.Generator().manual_seed(chunk)
    K = torch.randn((2, chunk, 128), generator=gen)
    if keys != "normal":
        K[:] = K[:, :1].clone()
    if keys == "halves":
        K[:, chunk // 2:] *= -0.5
    K = K.to(torch.bfloat16)
    for q in (0.001, 0.5, 0.9, 1.0):
        for seg_map, kind in ((MAP_LOGIT, O.MAP_LOGIT), (MAP_SOFTMAX, O.MAP_SOFTMAX)):
            ctx = LtriContext(config_from_workload(w, n_layers=1, theta=99.0, theta_quantile=q, seg_map=seg_map,
                                                   max_spans=1024), gpu_device)
            ka, _ = ctx.arena_views()
            ka[0, 0, :, :chunk].copy_(K)
            ctx.append_chunk(0, 0, 1, chunk)
            for h in range(2):
                M = O.chunk_map(K[h].double().numpy(), None, kind)[0]
                want = O.map_quantile(M, float(np.float32(q)))
                got = ctx.get_theta(0, 0, h)
                assert abs(got - want) <= 1e-5 * max(1.0, float(np.abs(np.tril(M)).max())), (q, seg_map, h, got, want)
