"""The rule that shapes a launch of the matrix-core attention (key groups per workgroup, splits of the key range), as the
library's host code has it."""
import os
import random
import shutil
import subprocess

import pytest

import __graft_entry__ as build_entry

PROGRAM = r"""
#include <stdio.h>
#include "attend_shape.h"
int main() {
  int hq, hkv, seqs, rows, ctx;
  long long part;
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

    def run(launches):
        text = "\n".join(" ".join(str(v) for v in x) for x in launches)
        out = subprocess.run([str(d / "a")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


def test_launches_that_one_group_serves_best_keep_it(shapes):
    """Measured at 32 query and 8 KV heads: two groups (2052 context tokens) or two groups and two splits (12292) took 1 to
    5 % longer here than one group without splits. (The last number: room as in a context of long chunks.)"""
    launches = [(32, 8, 1, rows, ctx, -1) for rows, ctx in
                [(1900, 2052), (2048, 2052), (1100, 12292), (1200, 12292), (1400, 12292), (1536, 12292), (2048, 12292)]]
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
