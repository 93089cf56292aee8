"""Blocks of a layer's eviction in one launch: each repeats its head's choice, so they leave part of the chip to other streams."""
import subprocess

import numpy as np
import pytest

from paper_2605_06676_amd import build as B

PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "lkv_shares.h"
int main(int n, char** v) {
  std::vector<int32_t> b;
  int64_t total = 0;
  const int n_seq = atoi(v[1]), stride = atoi(v[2]), heads = atoi(v[3]);
  for (int i = 5; i < n; ++i) b.push_back(atoi(v[i]));
  for (int i = 0; i < n_seq; ++i)
    for (int j = 0; j < heads; ++j) total += b[i * stride + j];
  int blocks = 0;
  const int rows = lkv::share_rows(b.data(), n_seq, stride, heads, total, atoi(v[4]) != 0, &blocks);
  printf("%d %d\\n", rows, blocks);
}
"""


@pytest.fixture(scope="module")
def shares(tmp_path_factory):
    d = tmp_path_factory.mktemp("shares")
    (d / "shares.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", B.CSRC, str(d / "shares.cpp"), "-o", str(d / "shares")], check=True)

    def run(budgets, heads, long_heads):
        n_seq, stride = budgets.shape
        args = [str(x) for x in (d / "shares", n_seq, stride, heads, int(long_heads))] + [str(int(x)) for x in budgets.reshape(-1)]
        rows, blocks = map(int, subprocess.run(args, check=True, capture_output=True, text=True).stdout.split())
        mine = budgets[:, :heads]
        if rows:      # the blocks that the kernel deals out
            assert blocks == np.maximum(1, -(-mine // rows)).sum()
        return rows, blocks

    return run


@pytest.mark.parametrize("kind", ["even", "one", "random", "zeros"])
@pytest.mark.parametrize("n_seq,heads,others", [(1, 1, 0), (1, 2, 6), (1, 4, 0), (2, 2, 3), (1, 5, 0), (1, 8, 8), (2, 8, 0), (1, 32, 0), (4, 16, 5)])
@pytest.mark.parametrize("total", [1, 64, 700, 5000, 39320, 52000, 120000, 400000])
def test_blocks(shares, n_seq, heads, others, total, kind):
    rng = np.random.default_rng(total + heads)
    n = n_seq * heads
    if kind == "even":
        b = np.full(n, total // n)
    elif kind == "one":
        b = np.full(n, 1 if total > n else 0)
        b[n // 2] = max(total - n, 1)
    elif kind == "random":
        b = rng.multinomial(total, rng.dirichlet(np.full(n, 0.3)))
    else:
        b = np.where(np.arange(n) % 2 == 0, total // n, 0)
    budgets = np.zeros((n_seq, heads + others), np.int64)
    budgets[:, :heads] = b.reshape(n_seq, heads)
    budgets[:, heads:] = 1000      # of other layers: none of this call's
    most = 128 if n <= 4 else 176
    for long_heads, limit in ((False, 300), (True, 900)):
        rows, blocks = shares(budgets, heads, long_heads)
        least = max(64, -(-int(b.sum()) // most))       # no share is smaller
        if rows == 0:
            assert np.maximum(1, -(-b // limit)).sum() > most
        else:
            assert least <= rows <= limit and blocks <= most
            if rows > 64:      # and one row fewer would take more blocks
                assert np.maximum(1, -(-b // (rows - 1))).sum() > most
