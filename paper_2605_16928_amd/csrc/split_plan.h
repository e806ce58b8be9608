// The split length of a selected-token plan (attn_decode.hip), apart so that it also compiles for the host.
#pragma once

namespace rtp {

// Shortest item, in blocks of 128 tokens (one round of loads): 5, since shorter items spend their time in the prologue and the
// merge -- but no longer than it takes to give one item to each of 256 compute units: with fewer, the launch lasts as long as
// the rounds of one item --, and no shorter than what leaves the longest unit 64 partials: one workgroup merges them all,
// eight at a time.  Both launches, us, items of 640 / one per compute unit / this: 12 rows of 4096 tokens 17.3 / 13.0 / 12.9, 32 of
// 1500 17.2 / 12.6 / 12.3, 1 of 8192 15.7 / 13.3 / 12.9; 1 of 16384 16.7 / 18.0 / 14.4, of 32768 19.5 / 27.4 / 17.3, of 65536 24.3 / 30.9 / 23.9,
// 2 of 16384 17.4 / 18.7 / 15.1, of 40000 23.2 / 24.5 / 22.7.
constexpr int kMinSplitBlocks = 5, kFewItems = 256, kFewPartials = 64;

__host__ __device__ __forceinline__ int at_most(int a, int b) { return a < b ? a : b; }
__host__ __device__ __forceinline__ int at_least(int a, int b) { return a > b ? a : b; }

// Blocks of 128 tokens per item: `total128` blocks in all units together, `longest128` in the longest, at most `target` items and
// one more per unit.
__host__ __device__ __forceinline__ int split_blocks(int total128, int longest128, int target) {
  const int shortest = at_least((total128 + kFewItems - 1) / kFewItems, (longest128 + kFewPartials - 1) / kFewPartials);
  target = at_least(target, 1);
  return at_least(at_least((total128 + target - 1) / target, at_most(kMinSplitBlocks, shortest)), 1);
}

}  // namespace rtp
