"""Block-to-work arithmetic of the one-block-per-head launches, compiled for the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2406_02542_amd", "csrc")
MAIN = r'''
#include <cstdio>
#include "block_order.h"
int main() {
  for (int n = 1; n <= 64; ++n) {
    printf("rank %d", n);
    for (int pos = 0; pos < n + 16; ++pos) printf(" %d", loki::paired_rank(pos, n));
    printf("\n");
  }
  const int groups[] = {2, 4, 8};
  for (int G : groups)
    for (int units = 1; units <= 40; ++units) {
      printf("slot %d %d", G, units);
      for (int b = 0; b < (units + 7) / 8 * 8 * G; ++b) printf(" %d:%d", loki::grouped_slot(b, G, units), loki::grouped_head(b, G));
      printf("\n");
    }
}
'''


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    cxx = shutil.which("g++")
    assert cxx, "g++ is part of the toolchain"
    d = tmp_path_factory.mktemp("order")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)
    return subprocess.run([str(d / "main")], check=True, capture_output=True, text=True).stdout.splitlines()


def test_every_sequence_has_one_place_and_no_other_place_has_one(lines):
    for line in (l.split() for l in lines if l.startswith("rank")):
        n, ranks = int(line[1]), [int(x) for x in line[2:]]
        assert sorted(ranks[:n]) == list(range(n))
        assert all(r == -1 for r in ranks[n:]), n


def test_blocks_of_a_padded_launch_cover_every_head_once(lines):
    for line in (l.split() for l in lines if l.startswith("slot")):
        G, units = int(line[1]), int(line[2])
        work = [tuple(int(v) for v in x.split(":")) for x in line[3:]]
        real = [w for w in work if w[0] >= 0]
        assert sorted(real) == [(u, g) for u in range(units) for g in range(G)]
        # a unit's heads go to one of the 8 dies, one after the other
        where = {w: b for b, w in enumerate(work) if w[0] >= 0}
        assert all(where[(u, g)] - where[(u, 0)] == 8 * g for u in range(units) for g in range(G))
