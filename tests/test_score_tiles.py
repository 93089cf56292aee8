"""Rows per block of the MLP scorer's launches: the rounds of blocks that the chip holds at once are not left half empty."""
import os
import subprocess

import pytest

from paper_2605_06676_amd import build as B

PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "lkv_tiles.h"
int main(int n, char** v) {
  std::vector<int32_t> lengths;
  for (int i = 3; i < n; ++i) lengths.push_back(atoi(v[i]));
  printf("%d\\n", lkv::score_mlp_rows_per_block(lengths.data(), (int)lengths.size(), atoll(v[1]), atoi(v[2])));
}
"""


@pytest.fixture(scope="module")
def rows_per_block(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    (d / "tiles.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", B.CSRC, str(d / "tiles.cpp"), "-o", str(d / "tiles")], check=True)

    def run(heads, hidden, lengths):
        args = [str(d / "tiles"), str(heads), str(hidden)] + [str(x) for x in lengths]
        rows = int(subprocess.run(args, check=True, capture_output=True, text=True).stdout)
        assert 256 <= rows <= 4096 and rows % 64 == 0
        return rows

    return run


def blocks(heads, lengths, rows):
    return sum(heads * -(-T // rows) for T in lengths)


@pytest.mark.parametrize("hidden", [16, 32, 48, 64, 96, 128])
@pytest.mark.parametrize("heads,lengths", [
    (288, [8192]), (288, [4096] * 2), (640, [4096]), (288, [32768]), (288, [4096]), (112, [65536]), (112, [20000]),
    (360, [3000]), (256, [32768]), (256, [131072]), (72, [16384]), (96, [32768]), (320, [6000]), (36, [120411]), (288, [2048]),
])
def test_sequences_of_one_length_fill_their_rounds(rows_per_block, heads, lengths, hidden):
    rows, chip = rows_per_block(heads, hidden, lengths), 1024 if hidden > 64 else 512
    rounds = -(-blocks(heads, lengths, rows) // chip)
    # rows the rounds have room for, against the rows there are (two prompts of 4096 over 288 heads as 576 blocks: 1.78)
    assert rounds * chip * rows <= 1.3 * heads * sum(lengths), (rows, rounds)


@pytest.mark.parametrize("hidden", [32, 64, 128])
@pytest.mark.parametrize("heads,lengths", [(8, [1]), (1, [70000]), (8, [17, 3000, 9001]), (8, [10001, 6214, 2491]), (64, [10001, 6214, 2491]),
                                           (5, [131072, 1]), (3, [2 ** 31 - 1]), (1024, [2 ** 21] * 32), (256, [1128, 245])])
def test_other_lengths(rows_per_block, heads, lengths, hidden):
    rows, chip = rows_per_block(heads, hidden, lengths), 1024 if hidden > 64 else 512
    n = blocks(heads, lengths, rows)
    if n <= 256:          # one to each compute unit, and no longer than it need be
        assert rows == 256 or blocks(heads, lengths, rows - 64) > 256
    else:                 # nor here: one tile less would take another round
        assert rows == 256 or -(-blocks(heads, lengths, rows - 64) // chip) > -(-n // chip) or len(set(lengths)) == 1
