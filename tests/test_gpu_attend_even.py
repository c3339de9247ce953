"""The attention in even shares (blocks strung together and cut anywhere, partial results folded in by the workgroup with a
block's last stage): rows and heads against the fp64 reference and a count of keys, at launches that the rule gives it."""
import shutil
import subprocess

import pytest
import torch

import __graft_entry__ as build_entry
from paper_2412_04757_amd import LtriContext, config_from_workload
from tests.test_gpu_attend_shapes import BF16_ROW, attend_reference, worst_row
from workloads import Workload, planted_stream, theta_default

# (query heads, KV heads, window, budget, history of each sequence, query rows)
LAUNCHES = [
    (32, 8, 1024, 1024, [4096], 1050),
    (32, 8, 1024, 4096, [8000], 1217),                 # two groups of keys or one, a ragged list
    (24, 2, 1024, 2048, [6000], 1500),                 # three workgroups per KV head
    (8, 8, 1024, 1024, [3000, 2500, 4000, 3500], 1092),  # one query head per KV head, four sequences, eight ragged row sub-tiles
    (32, 8, 1024, 1024, [3000, 2500, 2700], 336),      # two groups of keys, three sequences
    (16, 8, 1024, 2048, [5000, 3000, 700], 750),       # sequences of different lengths
    (32, 8, 1024, 1024, [4096, 1, 4096], 700),         # one of them without a context
]
# the rule leaves these alone: same checks, ordinary shapes
ORDINARY = [
    (8, 8, 1500, 4096, [9000, 9000], 2048),
    (32, 8, 300, 300, [2100] * 4, 600),
    (32, 8, 1024, 1024, [0, 0], 1121),                 # a first chunk
]
RULE = r"""
#include <stdio.h>
#include <algorithm>
#include "attend_shape.h"
using namespace ltri;
int main() {
  int hq, hkv, seqs, rows, ctx;
  while (scanf("%d %d %d %d %d", &hq, &hkv, &seqs, &rows, &ctx) == 5) {
    // the room that a context of as many sequences, chunks of 2048 and this many context tokens has
    const size_t row = 130 * sizeof(float), even = (attend_most_even_bytes(hq, hkv, seqs, 2048, 256) + row - 1) / row;
    const size_t room = std::max({(size_t)seqs * hq * ATT_MAX_SPLITS * ATT_SPLIT_MAX_ROWS, even, attend_most_part_rows(hq, hkv, seqs, 2048, ctx, 256)});
    printf("%d\n", attend_even(hq, hkv, seqs, rows, ctx, room * row, std::min(room, ATT_PART_MAX_ROWS), 256));
  }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("even")
    (d / "a.cpp").write_text(RULE)
    subprocess.run(["g++", "-O1", "-I" + build_entry.CSRC, str(d / "a.cpp"), "-o", str(d / "a")], check=True)

    def run(launches):
        text = "\n".join(" ".join(str(v) for v in x) for x in launches)
        return [int(v) for v in subprocess.run([str(d / "a")], input=text, capture_output=True, text=True, check=True).stdout.split()]
    return run


def test_even_shares_are_taken_where_the_chip_would_idle(rule):
    """The launches below, and those measured: never at a full chip or one that merely starts with idle units."""
    as_launched = lambda launches: [(hq, hkv, len(h), rows, min(max(h), 4 + window + budget)) for hq, hkv, window, budget, h, rows in launches]
    got = rule(as_launched(LAUNCHES))
    assert all(got) and got.count(1) >= 2 and got.count(2) >= 2, got
    assert got[[x[:2] for x in LAUNCHES].index((8, 8))] == 1
    assert rule(as_launched(ORDINARY)) == [0] * len(ORDINARY)
    assert rule([(32, 8, 1, 2048, 12292), (32, 8, 1, 1024, 8196), (32, 8, 1, 700, 2052), (32, 8, 4, 256, 2052), (8, 8, 1, 1024, 4100),
                 (32, 8, 1, 1800, 12292), (32, 8, 1, 128, 2052)]) == [0] * 7
    assert all(rule([(32, 8, 1, 1100, 8196), (32, 8, 1, 1300, 12292), (32, 8, 3, 700, 2052), (32, 8, 1, 700, 12292)]))
    # chunks without much of a context: in even shares they took 1.3 to 1.8 times as long
    assert rule([(32, 8, 2, 1121, 0), (16, 1, 4, 1397, 0), (32, 4, 2, 1574, 0), (24, 2, 3, 1097, 100), (8, 2, 6, 1809, 100), (64, 8, 3, 907, 0),
                 (24, 2, 2, 1443, 260), (32, 8, 4, 1956, 260), (16, 1, 16, 1033, 516)]) == [0] * 9


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,window,budget,history,rows", LAUNCHES + ORDINARY)
def test_even_shares(gpu_device, hq, hkv, window, budget, history, rows):
    S, longest = len(history), max(history)
    w = Workload("even", hq, hkv, 128, "bf16", longest + rows, 2048, 4, window, 0, budget, "uniform", 16, 96)
    ctx = LtriContext(config_from_workload(w, theta=theta_default(128), n_layers=1, n_seqs=S), gpu_device)
    ka, va = ctx.arena_views()
    q = []
    for s in range(S):
        K, V, Q, _ = planted_stream(w, 300 + s, device=str(gpu_device), context=longest + rows)
        ka[0, s].copy_(K)
        va[0, s].copy_(V)
        q.append(Q[:rows])
        for c0 in range(0, history[s], 1000):
            ctx.append_chunk(0, s, 1, min(1000, history[s] - c0))
    q = torch.stack(q).contiguous()
    ctx.append_chunk(0, 0, S, rows)
    ctx.retrieve(0, 0, S, q)
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device=gpu_device)
    out = ctx.attend(0, 0, S, q, lse=lse)
    for _ in range(3):                                   # the flags are left as they were found
        again = torch.full_like(q, float("nan"))
        ctx.attend(0, 0, S, q, out=again)
        assert torch.equal(out, again)
    ctx.set_attend_stages(3)                             # the shorter ring: same results
    ctx.attend(0, 0, S, q, out=again.fill_(float("nan")))
    assert torch.equal(out, again)
    ctx.set_attend_stages(4)
    for s in range(S):
        want, want_lse = attend_reference(ctx, w, s, history[s], q[s])
        assert worst_row(out[s], want) <= BF16_ROW
        assert float((lse[s].double() - want_lse).abs().max()) <= 2e-3
    # equal weights: an output times the number of keys counts the keys of a column (bf16 holds a hundred or so), the
    # log-sum-exp is the logarithm of their number
    gen = torch.Generator(device=gpu_device).manual_seed(21)
    column = torch.randint(0, 128, va.shape[:-1], generator=gen, device=gpu_device)
    ka.zero_(), va.zero_()
    va.scatter_(-1, column.unsqueeze(-1), 1.0)
    out = ctx.attend(0, 0, S, q, lse=lse).double()
    G = hq // hkv
    for s in range(S):
        for h in range(hkv):
            t = torch.from_numpy(ctx.get_token_list(0, s, h)).long().to(gpu_device)
            one = torch.nn.functional.one_hot(column[0, s, h], 128).double()
            count = one[t].sum(0) + one[history[s]:history[s] + rows].cumsum(0)
            n = count.sum(1)
            assert float(count.max()) < 120
            got = out[s, :, h * G:(h + 1) * G] * n[:, None, None]
            assert bool(((got - count[:, None]).abs() <= 2.0 ** -8 * count[:, None]).all())
            assert float((lse[s, :, h * G:(h + 1) * G].double() - n.log()[:, None]).abs().max()) <= 2e-6
    assert ctx.sync_status() == 0
