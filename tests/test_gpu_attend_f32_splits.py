"""The fp32 attention with its key range split over workgroups, the last of which to finish a tile of (row, head) pairs adds the
splits up: against the fp64 reference, at launches that split, and where splits have no key."""
import shutil
import subprocess

import pytest
import torch

import __graft_entry__ as build_entry
from paper_2412_04757_amd import LtriContext, config_from_workload
from tests.test_gpu_attend_shapes import attend_reference
from workloads import Workload, planted_stream, theta_default

# (query heads, KV heads, head_dim, sequences, window, k_max, budget, history, query rows), splits
LAUNCHES = [
    ((4, 2, 128, 2, 300, 0, 300, 1500, 37), 2),        # two sequences and KV heads, a last workgroup of 10 pairs
    ((6, 2, 64, 2, 500, 0, 300, 1500, 85), 3),         # a group of three heads, its last workgroup ragged
    ((2, 1, 128, 1, 600, 0, 600, 2500, 100), 4),       # both column parts
    ((12, 4, 64, 1, 500, 0, 600, 2500, 70), 4),
    ((4, 1, 64, 1, 900, 0, 600, 2500, 1), 4),          # one row, four pairs
    ((40, 2, 128, 3, 900, 0, 200, 2500, 3), 4),        # 60 pairs of 20 heads
    ((4, 1, 64, 1, 64, 4, 0, 1500, 9), 4),             # shaped for four long spans; the spans are short, and two splits have no key
    ((8, 2, 128, 2, 40, 4, 0, 1500, 20), 4),
]
RULE = r"""
#include <stdio.h>
#include "attend_shape.h"
int main() {
  int g, hkv, seqs, rows, ctx;
  while (scanf("%d %d %d %d %d", &g, &hkv, &seqs, &rows, &ctx) == 5) printf("%d\n", ltri::attend_f32_splits(g, hkv, seqs, rows, ctx));
}
"""


def test_these_launches_split(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    (tmp_path / "a.cpp").write_text(RULE)
    subprocess.run(["g++", "-O1", "-I" + build_entry.CSRC, str(tmp_path / "a.cpp"), "-o", str(tmp_path / "a")], check=True)

    def splits(launches):
        text = "\n".join(" ".join(str(v) for v in x) for x in launches)
        return [int(v) for v in subprocess.run([str(tmp_path / "a")], input=text, capture_output=True, text=True, check=True).stdout.split()]
    # (a span counts as 256 tokens where only their number is limited)
    got = splits([(hq // hkv, hkv, S, rows, min(history, 4 + window + (budget or 256 * k))) for (hq, hkv, _, S, window, k, budget, history, rows), _
                  in LAUNCHES])
    assert got == [n for _, n in LAUNCHES]
    # a full round of workgroups, a short list, and the last sizes on either side of a limit (64 | 65 workgroups, 512 | 496 keys)
    assert splits([(4, 1, 4, 256, 5000), (4, 1, 1, 256, 100), (4, 1, 1, 256, 5000), (4, 1, 1, 260, 5000), (4, 1, 1, 16, 496), (4, 1, 1, 16, 480)]) \
        == [1, 1, 4, 3, 2, 1]


@pytest.mark.gpu
@pytest.mark.parametrize("launch,splits", LAUNCHES)
def test_fp32_attention_in_splits(gpu_device, launch, splits):
    hq, hkv, dim, S, window, k_max, budget, history, rows = launch
    w = Workload("f32-splits", hq, hkv, dim, "f32", history + rows, 256, 4, window, k_max, budget, "uniform", 8, 24)
    ctx = LtriContext(config_from_workload(w, theta=theta_default(dim), n_layers=1, n_seqs=S), gpu_device)
    ka, va = ctx.arena_views()
    q = []
    for s in range(S):
        K, V, Q, _ = planted_stream(w, 900 + s, device=str(gpu_device), context=history + rows)
        ka[0, s].copy_(K), va[0, s].copy_(V)
        q.append(Q[history:])
    # spans of 20 tokens, given: their number limits the retrieved tokens
    for s in range(S):
        for c0 in range(0, history, 240):
            n = min(240, history - c0)
            ctx.append_chunk_with_spans(0, s, n, [sorted({*range(0, n, 20), n})] * hkv)
    q = torch.stack(q).contiguous()
    ctx.append_chunk(0, 0, S, rows)
    ctx.retrieve(0, 0, S, q)
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device=gpu_device)
    out = torch.full_like(q, float("nan"))
    ctx.attend(0, 0, S, q, out=out, lse=lse)
    for _ in range(3):                                   # the counters are left as they were found
        again, lse_again = torch.full_like(q, float("nan")), torch.full_like(lse, float("nan"))
        ctx.attend(0, 0, S, q, out=again, lse=lse_again)
        assert torch.equal(out, again) and torch.equal(lse, lse_again)
    for s in range(S):
        if k_max:                                        # tiles of 16 keys go round 8 wavefronts of each split: the last splits get none
            assert len(ctx.get_token_list(0, s, 0)) + rows <= 16 * 8 * (splits - 2)
        want, want_lse = attend_reference(ctx, w, s, history, q[s])
        # as for launches without splits: scores of up to 128 fp32 products of values around 1 and |score| <= 8 are off by
        # 128 * 2^-24 * 8 at the very most in the exponent; a split more adds one rounding of sums and weights (2^-23)
        assert float((out[s].double() - want).abs().max()) <= 6e-5
        assert float((lse[s].double() - want_lse).abs().max()) <= 6e-5
    assert ctx.sync_status() == 0
