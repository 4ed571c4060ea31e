// How the projections and the one-launch fp32 kernel split their work into blocks.  Plain C++ with no GPU dependency, so that the
// rules can be tested on a machine without a GPU.
#pragma once
#include <algorithm>

namespace aa {

// --- projections (projection_kernel): rows of X and outputs a block, channels a step; M rows, O outputs, K channels ---
struct ProjectionBlocks {
  int rows, outputs, step;
};
inline ProjectionBlocks projection_blocks(long long M, int O, int K, int compute_units) {
  const long long bytes = 2 * M * (K + O);      // of X and Y
  // Channels per step: 64 ask for whole 128-byte lines (16384 rows, width 512: 41.7 us, 47.0 with steps of 32).  32 where four to
  // five blocks a CU do more: up to a width of 96 (100352 rows, width 96: 18.7 us, 22.5 with steps of 64), and below 256 where
  // the last 64 would be half empty (width 160: 32.4, 38.2) or from memory (100352 rows, width 192: 50.8 + 20.5, 52.9 + 21.8;
  // 25088 rows: 17.1 + 7.9, 15.5 + 7.5).
  const int step = K < 128 || (K < 256 && ((K - 1) % 64 < 32 || bytes > (64ll << 20))) ? 32 : 64;
  // Rows per block: 64 while blocks of 128 would leave CUs at less than half of what they hold (784 rows, width 512: 11.1 ->
  // 9.0 us; 6272 rows, output of width 512: 10.0 -> 8.4; but q | k | v of width 256, 294 blocks: 10.2, 12.2 with 64 rows), and
  // where two a CU leave a few for a second round, for which three blocks of 64 rows a CU are shorter (14 products of 517 to
  // 588 blocks of 128 rows 0.85 to 0.97 of the time: 18000 rows, width 512, output 18.4 -> 16.6).
  const long long tall = (M + 127) / 128 * ((O + 127) / 128), cus = compute_units;
  const bool low = step == 32 ? tall < 2 * cus : tall < cus || (tall > 2 * cus && tall <= 5 * cus / 2);
  // Outputs per block: the least padded width, an output of a narrower block priced higher: it takes 8 / 12 (96) or 6 / 8 (64)
  // LDS reads per product where 128 takes 8 / 16.  (64 are the cheapest up to 64 outputs alone, of as many channels at most.)
  auto price = [&](int outputs, int each) { return (long long)((O + outputs - 1) / outputs) * outputs * each; };
  const long long p128 = price(128, 10), p96 = price(96, 12), p64 = step == 32 ? price(64, 13) : p128;
  const int outputs = p128 <= p96 && p128 <= p64 ? 128 : p96 <= p64 ? 96 : 64;
  // X and Y beyond three quarters of the 256 MB that caches keep: the loads are longer under way, and blocks of 256 rows with
  // two steps of 32 channels ahead do better.  100352 rows, q | k | v of width 256: 81.5 us in the blocks below, 75.8; of
  // 384: 149, 138.5; 25088 rows, width 1024: 200, 188; but width 768 (147 MB): 115, 116 to 123.
  if (outputs == 128 && !low && step == 64 && bytes > (192ll << 20)) return {256, 128, 32};
  return {low ? 64 : 128, outputs, step};
}

// --- fp32 units in one launch (fused_f32_kernel) ---
// Blocks per unit: while CUs are idle, further blocks repeat what comes before the broadcast and share out its tiles of 16 tokens,
// down to one per SIMD, and the channels of V, one 16-channel tile each (or two of four).  The same sums in the same order.
// 1 unit of 196 tokens x 49 agents, d = 32: 15.0 us in one block, 11.8 in four, 10.5 in eight (tiles and channels).
struct UnitShares {
  int tiles, parts, channel_tiles;      // tiles of tokens a block takes at most, blocks along them, 16-channel tiles a block takes
};
inline UnitShares fused_f32_shares(int N, int d, int units, int compute_units) {
  const int ntiles = (N + 15) / 16, dt = (d + 15) / 16;
  const int tiles = (ntiles - 1) / std::max(1, std::min((ntiles + 3) / 4, compute_units / units)) + 1;
  const int parts = (ntiles - 1) / tiles + 1;
  int ct = 1;
  while (ct < dt && (dt % ct != 0 || dt / ct * parts * units > compute_units)) ++ct;
  return {tiles, parts, ct};
}

}  // namespace aa
