"""The word by which a workgroup of the attention's even shares hands its partial result to another: every order of the giver's one
and the taker's several steps leaves it at zero for the next launch, and a result is folded in exactly when it is there."""
import shutil
import subprocess

import pytest

import __graft_entry__ as build_entry

# The giver comes after `when` steps of the taker, which are counted as it makes them; twice over the same word.
PROGRAM = r"""
#include <stdio.h>
#include "handoff.h"
struct Shared { int word, step, when; bool given; };
struct Word {
  Shared* s;
  void tick() const {
    if (s->step++ == s->when) { s->given = true; s->word += 1; }        // what handoff_give does (checked in main)
  }
  int load() const { tick(); return s->word; }
  void store(int v) const { tick(); s->word = v; }
  int add(int v) const { tick(); const int old = s->word; s->word += v; return old; }
  void pause() const { tick(); }
};
int main() {
  Shared g{0, 0, -1, false};
  ltri::handoff_give(Word{&g});
  printf("%d\n", g.word);
  for (int polls = 0; polls < 5; ++polls)
    for (int when = 0; when < 14; ++when) {
      Shared s{0, 0, when, false};
      for (int launch = 0; launch < 2; ++launch) {
        const bool took = ltri::handoff_take(Word{&s}, polls);
        const bool there = s.given;
        if (!s.given) s.word += 1;                                       // the giver comes once the taker has gone
        printf("%d %d %d %d %d\n", polls, when, took, there, s.word);
        s.step = 0; s.given = false;
      }
    }
}
"""


def test_no_order_of_events_leaves_a_word_behind(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    (tmp_path / "a.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-I" + build_entry.CSRC, str(tmp_path / "a.cpp"), "-o", str(tmp_path / "a")], check=True)
    lines = subprocess.run([str(tmp_path / "a")], capture_output=True, text=True, check=True).stdout.splitlines()
    assert lines[0] == "1" and len(lines) == 1 + 5 * 14 * 2
    gave_up = 0
    for line in lines[1:]:
        polls, when, took, there, word = (int(v) for v in line.split())
        assert took == there and word == 0, line
        gave_up += not took
    assert 0 < gave_up < len(lines) - 1
