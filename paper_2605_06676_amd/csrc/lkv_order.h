// Order of the blocks of a causal attention launch (plain C++).
#pragma once

namespace lkv {

// Query tile and head of a block in a causal attention grid of n_tiles * n_heads blocks of 256 threads, two to a
// compute unit, whose work grows with the tile.  In order of decreasing work (tile slow, head fast), but block i and block
// i + 256 of a launch start on one compute unit and share it (read from the hardware's id registers), so of the first
// 512 the second half comes in increasing order: the longest with the shortest.  Below 512 blocks the longest have a compute
// unit to themselves.  Block i runs on XCD i mod 8: where the heads divide by 8 each XCD takes neighbouring ones, which
// share their KV head's rows in its L2.  Forward, in turn with plain decreasing order: 32 heads of 1500 tokens 36.6 ->
// 34.7 us, 2345 62.7 -> 59.5, 4096 149 -> 144, 6000 296 -> 294, 16384 2044 -> 2042; 8 heads of 9000 198 -> 190; 28 heads of
// 2048 48.0 -> 44.7, 9000 568 -> 572.
constexpr int kComputeUnits = 256;
struct CausalBlock {
  int tile, head;
};
constexpr CausalBlock causal_block(int block, int n_tiles, int n_heads) {
  const int paired = n_tiles * n_heads < 2 * kComputeUnits ? n_tiles * n_heads : 2 * kComputeUnits;
  const int shared = paired - kComputeUnits;   // compute units that start with two blocks, if any
  int rank = block;
  if (shared > 0 && block < paired) {
    if (block >= kComputeUnits) rank = paired - 1 - (block - kComputeUnits);
    else rank = block < shared ? block + kComputeUnits - shared : block - shared;
  }
  int head = rank % n_heads;
  if (n_heads % 8 == 0) head = (head & 7) * (n_heads >> 3) + (head >> 3);
  return {n_tiles - 1 - rank / n_heads, head};
}

}  // namespace lkv
