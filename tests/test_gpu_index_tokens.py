"""Index tokens of dynamic index vectors at the span lengths where the ranking of a span's tokens changes method, and
under budgets per memory block that several wavefront passes of spans share."""
import numpy as np
import pytest
import torch

from oracle import ltri_oracle as O
from paper_2412_04757_amd import LtriContext, config_from_workload
from workloads import Workload

pytestmark = pytest.mark.gpu


def cuts(lens, total, unit):
    b = np.concatenate([[0], np.cumsum(lens)])
    b = b[b < total]
    return np.unique(np.concatenate([b, [total], np.arange(0, total, unit) if unit else []]).astype(np.int64))


# (span lengths, repeated to fill the chunk; tokens; unit; index vectors per block)
CASES = [
    ([255, 256, 257, 1, 2, 63, 64, 65], 963, 0, 0),
    ([1], 256, 128, 12),               # more spans in a block than its budget, two per lane
    ([3, 1, 7, 2], 1024, 512, 200),    # 158 spans per block, levelled, with a remainder
    ([40, 9, 79], 900, 128, 12),
    ([500, 12], 1024, 512, 64),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_index_tokens_at_method_changes(gpu_device, case):
    lens, n, unit, block_max = CASES[case]
    H = 4
    b = cuts(np.resize(lens, n), n, unit)
    w = Workload("mini-index", 4, H, 128, "bf16", 1024, 1024, 4, 64, 4, 0, "uniform", 16, 128)
    ctx = LtriContext(config_from_workload(w, n_layers=1, theta=1e30, rep_mode=O.REP_DYNAMIC, lam=1.0, unit_tokens=unit,
                                           index_block_max=block_max, max_spans=1024), gpu_device)
    K = (0.35 * torch.randn((H, n, 128), generator=torch.Generator().manual_seed(case))).to(torch.bfloat16)
    ka, _ = ctx.arena_views()
    ka[0, 0, :, :n].copy_(K)
    ctx.append_chunk_with_spans(0, 0, n, [b] * H)
    audited = 0
    for h in range(H):
        Kh = K[h].double().numpy()
        A, _ = O.chunk_map(Kh, None, O.MAP_SOFTMAX)
        args = (A, b, 1.0, 1, 0, O.RATIO_ROW)
        if not O.dynamic_index_is_stable(*args, rel=2.0 ** -18, block_max=block_max, unit=unit, c0=0):
            continue                   # a near-tie that an fp32 map cannot decide the way fp64 does
        audited += 1
        want = O.dynamic_index_tokens(*args, block_max=block_max, unit=unit, c0=0)
        assert list(ctx.get_index_tokens(0, 0, h, n)) == list(np.concatenate(want)), h
        reps = O.index_vector_sums(Kh, want, "bf16")
        assert np.array_equal(ctx.get_rep_keys(0, 0, h).double().numpy(), reps), h
    assert audited >= 1
    assert ctx.sync_status() == 0
