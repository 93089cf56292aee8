// Shares of the blocks of a layer's eviction in one launch (plain C++).
#pragma once
#include <cstdint>

namespace lkv {

// Every block of the one-launch top-k and compaction makes its head's whole choice again before it copies its share of the
// rows.  On an idle chip that is free, beside other streams' work it is not: more blocks copy sooner, and cost a busy chip more.
// About two thirds of the compute units, and half of them for up to four heads (whose copies are short), is where a lone stream loses
// little, and two streams, or four, that evict layer after layer lose nothing against two launches (a block per head that chooses,
// the compaction behind it).  Two launches as they were : 256 blocks in all : 176 : 128 (the linear scorer, 32 layers of 32768 tokens, ms):
//   8 heads: one stream 1.67 : 1.46 : 1.48 : 1.54, two 1.27 : 1.30 : 1.22 : 1.19, four 1.34 : 1.38 : 1.32 : 1.30
//   4 heads: one stream 1.23 : 1.04 : 1.03 : 1.06, two 0.78 : 0.83 : 0.78 : 0.74, four 0.91 : 0.92 : 0.88 : 0.84
// Captured in a graph, where nothing but the chip bounds the streams, four of them still pay: a call over 8 heads 33.4 us in two
// launches, 38.2 : 35.9 : 34.2 here (alone 51.4, 44.2 : 45.3 : 46.9); over 8 of 131072 with a 256-64-1 scorer 115.6, 119.7 : 118.1 (alone
// 143.9, 136.2 : 138.6).
// A head that holds most of the rows has most of the blocks; the same weighing holds for it (8 heads of 32768, one with nearly all of 13
// thousand rows, scores given: alone 22.5, 16.1 : 16.0; two captured streams 14.6, 13.6 : 12.6; four 13.4, 12.8 : 11.4).
constexpr int kShareBlocks = 176;
constexpr int kShareBlocksFew = 128;
constexpr int kShareFewHeads = 4;

// Rows of a block at most.  With more of them the copy decides, and sixteen waves a compute unit copy more slowly than the
// compaction's blocks.  Two launches : 192 blocks, alone (us), linear scorer: 283 rows a block 52.0 : 50.3 (8 heads of 34000) and 72.8 :
// 72.2 (16), 425 56.4 : 56.3 and 77.1 : 78.4, 567 61.2 : 62.4; 64 heads of 8192, 273 62.7 : 62.1, 32 heads of 8192, 410 46.9 : 48.1.
// Heads too long for the registers, whose way through the two launches is longer: 8 heads of 131072, 819 rows 141.0 : 138.4, 1092
// 153.9 : 154.2; 16 of 60000, 750 rows 128.7 : 128.6, 1000 137.5 : 139.3.
constexpr int kShareRows = 300;
constexpr int kShareRowsLong = 900;

// Blocks that shares of up to `rows` rows make, one at least for each of n_seq * heads heads (budgets: of sequence i's head j at
// [i * seq_stride + j]).
inline int64_t share_blocks(const int32_t* budgets, int n_seq, int seq_stride, int heads, int64_t rows) {
  int64_t n = 0;
  for (int i = 0; i < n_seq; ++i)
    for (int j = 0; j < heads; ++j) {
      const int64_t parts = (budgets[(size_t)i * seq_stride + j] + rows - 1) / rows;
      n += parts > 1 ? parts : 1;
    }
  return n;
}

// Rows of a share (64 at least), and the blocks: as many as go with so many heads (at most 128 of them).  0 where that takes more
// rows than pay.
inline int share_rows(const int32_t* budgets, int n_seq, int seq_stride, int heads, int64_t total_rows, bool long_heads, int* blocks) {
  auto count = [&](int64_t rows) { return share_blocks(budgets, n_seq, seq_stride, heads, rows); };
  const int most = n_seq * heads <= kShareFewHeads ? kShareBlocksFew : kShareBlocks;
  int64_t lo = total_rows / most, hi = lo < 32 ? 64 : 2 * lo;   // hi is enough, lo is not
  if (lo < 63) lo = 63;
  while (count(hi) > most) hi *= 2;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) / 2;
    (count(mid) > most ? lo : hi) = mid;
  }
  if (hi > (long_heads ? kShareRowsLong : kShareRows)) return 0;
  *blocks = (int)count(hi);
  return (int)hi;
}

}  // namespace lkv
