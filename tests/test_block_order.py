"""The order in which a causal attention launch deals query tiles and heads to its blocks: every pair once, and compute
units that start with two blocks start with a long and a short one."""
import os
import subprocess

import pytest

from paper_2605_06676_amd import build as B

PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "lkv_order.h"
int main(int, char** v) {
  const int tiles = atoi(v[1]), heads = atoi(v[2]);
  for (int b = 0; b < tiles * heads; ++b) {
    const lkv::CausalBlock x = lkv::causal_block(b, tiles, heads);
    printf("%d %d\\n", x.tile, x.head);
  }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", B.CSRC, str(d / "order.cpp"), "-o", str(d / "order")], check=True)
    return str(d / "order")


@pytest.mark.parametrize("tiles,heads", [(1, 1), (3, 7), (32, 8), (257, 1), (37, 7), (12, 32), (511, 1), (16, 32), (19, 32), (128, 28), (1025, 4)])
def test_every_block_once_and_long_beside_short(program, tiles, heads):
    lines = subprocess.run([program, str(tiles), str(heads)], check=True, capture_output=True, text=True).stdout.split()
    got = list(zip(map(int, lines[::2]), map(int, lines[1::2])))
    assert sorted(got) == [(t, h) for t in range(tiles) for h in range(heads)]
    n = len(got)
    work = [t + 1 for t, _ in got]
    assert work[512:] == sorted(work[512:], reverse=True)
    first = sorted(work[:512], reverse=True)
    if n <= 256:
        assert work == first
    else:
        shared = min(n, 512) - 256
        load = [work[i] + (work[i + 256] if i < shared else 0) for i in range(256)]
        # at best the longest block alone, or the mean of a pair; dealt in plain decreasing order the first unit gets
        # the longest block and the 257th
        tail = first[256 - shared:]
        assert max(load) <= max(first[0], max(tail[i] + tail[-1 - i] for i in range(shared)))
