// Tiles of the MLP scorer's launches (plain C++).
#pragma once
#include <cstdint>

namespace lkv {

// Rows per block of a launch.  Every wave starts by loading the hidden layer's weights, and a last round that is a small part
// of one leaves the chip idle.
// Sequences of one length: the tiles for which the rounds of what the chip holds at once (512 blocks of four waves for hidden
// widths up to 64, 1024 of two), each as long as a tile and 128 rows, come out shortest.  As few blocks as fill whole rounds,
// however long they get, are not it where the heads do not divide a round: two prompts of 4096 tokens over 288 heads went out as
// 576 blocks of 4096 rows and took 249 us at width 64 and 292 at 128, where 1024 and 832 rows take 213 and 240 (and one
// of 8192 226, where 1664 take 215).  Two corrections, both measured: tiles of 2048 rows and more that divide the sequence count
// for less (288 heads of 32768 tokens, width 128: 2368 rows 874 us, 2048 862), and widths that leave the matrix units room (up
// to 48, and up to 96) are bound by the stream, where blocks of more than 1024 rows are slower once they go round several times (256
// heads of 32768, width 96: 2048 rows 747, 4096 786, 1024 707).
// Sequences of unlike lengths even a round out among themselves, the longest first: as few blocks as fill whole rounds
// (three of 14336, 8923 and 3574 tokens over 8 heads, width 64: 24.2 us; by the rule above, whose tiles would be
// shorter, 26.8).
// Few rows go one block to each of the 256 compute units, as long as these have up to 1280 rows (384 of the two-wave blocks): a
// second block on some of them would take as long as one on all.
// Against tiles of a power of two for each length, launched apart where they differ, 110 drawn sizes of 16 to 128 units: 1.09
// times as fast in the mean, all but four between 0.98 and 1.43 (three lengths over 288 heads, 128 units, 0.96; three of 12288
// tokens over 144 heads, 64 units, 0.95: a twelfth of a round more than three or ten).  Width 64: 8
// heads, sequences of 10001, 6214 and 2491 tokens 26.6 -> 17.6 us, 70 of 9001 643 -> 470, one of 32768 28.2 -> 25.2; width
// 128: 40 of 2000 over 32 heads 314 -> 251, 36 heads of 120411 454 -> 404.
inline int score_mlp_rows_per_block(const int32_t* seq_len, int n_seq, int64_t heads, int hidden) {
  constexpr int kUnits = 256, kLeast = 256, kMost = 4096, kStep = 64;
  constexpr int kFixed = 128;                             // rows that a block's start takes as long as
  constexpr int kEven = 2048;                             // rows from which a tile that divides the sequence counts for less
  const int64_t round = hidden > 64 ? 1024 : 512;
  const int most_alone = hidden > 64 ? 384 : 1280;        // rows of a block that has its compute unit to itself
  const bool narrow = hidden <= 48 || (hidden > 64 && hidden <= 96);
  const int most_again = narrow ? 1024 : kMost;           // and of one in several rounds
  int64_t keys = 0;
  bool alike = true;
  for (int s = 0; s < n_seq; ++s) {
    keys += heads * seq_len[s];
    alike &= seq_len[s] == seq_len[0];
  }
  auto blocks = [&](int rows) {
    if (alike) return n_seq * heads * (((int64_t)seq_len[0] + rows - 1) / rows);
    int64_t n = 0;
    for (int s = 0; s < n_seq; ++s) n += heads * (((int64_t)seq_len[s] + rows - 1) / rows);
    return n;
  };
  auto rows_for = [&](int64_t limit, int most) {   // the least of at most `most` that give up to `limit` blocks
    const int64_t share = keys / limit / kStep * kStep;   // below this nothing does
    int rows = (int)(share < kLeast ? kLeast : share < most ? share : most);
    while (rows < most && blocks(rows) > limit) rows += kStep;
    return rows;
  };
  if (blocks(most_alone) <= kUnits) return rows_for(kUnits, most_alone);
  if (!alike) {
    const int most = blocks(kMost) > round ? most_again : kMost;
    return rows_for((blocks(most) + round - 1) / round * round, most);
  }
  int best = kMost;
  int64_t least = INT64_MAX;
  for (int rows = kLeast; rows <= kMost; rows += kStep) {
    const int64_t rounds = (blocks(rows) + round - 1) / round;
    if (rounds > 1 && rows > most_again) continue;
    const int64_t cost = rounds * (rows + kFixed) * (rounds > 1 && rows >= kEven && seq_len[0] % rows == 0 ? 29 : 32);
    if (cost <= least) { least = cost; best = rows; }
  }
  return best;
}

}  // namespace lkv
