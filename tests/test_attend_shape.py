"""The rule that shapes a launch of the matrix-core attention (key groups per workgroup, splits of the key range), as the
library's host code has it."""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

import __graft_entry__ as build_entry
from paper_2412_04757_amd import config_from_workload, load_library
from workloads import Workload

PROGRAM = r"""
#include <stdio.h>
#include "attend_shape.h"
int main(int argc, char**) {
  int hq, hkv, seqs, rows, ctx;
  long long part;
  if (argc > 1) {                              // most partial rows within a context's limits
    while (scanf("%d %d %d %d %d", &hq, &hkv, &seqs, &rows, &ctx) == 5)
      printf("%zu\n", ltri::attend_most_part_rows(hq, hkv, seqs, rows, ctx, 256));
    return 0;
  }
  while (scanf("%d %d %d %d %d %lld", &hq, &hkv, &seqs, &rows, &ctx, &part) == 6) {
    const ltri::AttShape s = ltri::attend_shape(hq, hkv, seqs, rows, ctx, rows, part < 0 ? ltri::ATT_PART_MAX_ROWS : (size_t)part, 256);
    printf("%d %d\n", s.ks, s.ns);
  }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("shape")
    (d / "a.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-I" + build_entry.CSRC, str(d / "a.cpp"), "-o", str(d / "a")], check=True)

    def run(launches, *mode):
        text = "\n".join(" ".join(str(v) for v in x) for x in launches)
        out = subprocess.run([str(d / "a"), *mode], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


def test_launches_that_one_group_serves_best_keep_it(shapes):
    """Measured at 32 and 64 query and 8 KV heads: two groups (2052 context tokens, none) or two groups and two splits (12292)
    took 1 to 7 % longer here than one group without splits. (The last number: room as in a context of long chunks.)"""
    launches = [(32, 8, 1, rows, ctx, -1) for rows, ctx in
                [(1900, 2052), (2048, 2052), (1100, 12292), (1200, 12292), (1400, 12292), (1536, 12292), (2048, 12292)]]
    launches.append((64, 8, 1, 2048, 0, -1))
    assert shapes(launches) == [(1, 1)] * len(launches)


def test_launches_that_leave_compute_units_idle_do_not(shapes):
    launches = [(32, 8, 1, 1024, 12292, -1), (32, 8, 4, 256, 2052, -1), (32, 8, 1, 512, 12292, -1), (32, 8, 1, 128, 2052, -1),
                (8, 8, 1, 300, 4100, -1), (8, 2, 1, 2048, 6148, -1)]
    assert all(ks * ns > 1 for ks, ns in shapes(launches))


def test_shapes_stay_within_what_the_kernels_take(shapes):
    rng = random.Random(4)
    launches = []
    for _ in range(4000):
        hkv = rng.choice([1, 2, 8])
        launches.append((hkv * rng.choice([1, 2, 4, 8, 12]), hkv, rng.randint(1, 64), rng.randint(5, 2048),
                         rng.randint(0, 20000), rng.choice([0, 100, 5000, 65536])))
    for (hq, hkv, seqs, rows, ctx, part), (ks, ns) in zip(launches, shapes(launches)):
        assert ks in (1, 2) and 1 <= ns <= 16
        assert ns == 1 or (seqs * hq * rows * ns <= part and ks * ns <= -(-ctx // 64) + -(-rows // 64))


def test_a_context_has_room_for_the_shapes_its_launches_take(shapes):
    """Partial results are sized by what attend_shape takes within the context's limits: launches inside them are shaped as
    if there was room for any (a few in a hundred, between the row counts and contexts that are looked at, may not be)."""
    rng = random.Random(5)
    for limits in [(32, 8, 1, 256, 2052), (32, 8, 4, 256, 2052), (32, 8, 1, 2048, 12292), (8, 8, 3, 700, 3000), (8, 2, 1, 512, 300)]:
        hq, hkv, seqs, chunk, ctx = limits
        room = shapes([limits], "room")[0][0]
        assert room <= 65536
        inside = [(hq, hkv, rng.randint(1, seqs), rng.randint(5, chunk), rng.randint(0, ctx)) for _ in range(1000)]
        got, free = shapes([x + (room,) for x in inside]), shapes([x + (-1,) for x in inside])
        assert sum(a == b for a, b in zip(got, free)) >= 970
    assert shapes([(8, 2, 1, 512, 300)], "room") == [(0,)]          # never split


@pytest.mark.parametrize("hq,hkv,seqs,chunk,window,budget,tokens,megabytes", [
    (32, 8, 1, 256, 1024, 1024, 8192, 24),        # 17 MB of partial results
    (8, 2, 1, 512, 96, 200, 1200, 4),             # blocks of up to four rows only
])
def test_scratch_of_contexts_that_split_little(hq, hkv, seqs, chunk, window, budget, tokens, megabytes):
    w = Workload("size", hq, hkv, 128, "bf16", tokens, chunk, 4, window, 0, budget, "uniform", 16, 96)
    cfg = config_from_workload(w, theta=1.0, n_layers=1, n_seqs=seqs)
    state, scratch = C.c_size_t(), C.c_size_t()
    assert load_library().ltri_workspace_bytes(C.byref(cfg), C.byref(state), C.byref(scratch)) == 0
    assert scratch.value < megabytes << 20
