// Which forward kernels take their tokens in columns (16 image columns of some image rows a wave) and which in rows (runs of
// consecutive tokens).  Plain C++ with no GPU dependency, so that the rules can be tested on a machine without a GPU.
#pragma once
#include <algorithm>

namespace aa {

// --- few agents (small_broadcast_cols_kernel), with a convolution ---
// Columns unless more than a third of the sixteens lie beside the image.  Whole forward, 96 units, n = 49, rows / columns in us:
// d = 32, 40 x 33 tokens 35.2 / 32.5, 48 x 28 35.2 / 31.7, 48 x 22 30.7 / 30.8, 64 x 17 30.6 / 31.6; d = 64, 56 x 56 112 / 88, 40 x 33
// 71.9 / 64.7, 48 x 22 56.5 / 56.8, 60 x 20 59.8 / 60.9.
// Rows of the output of 4 GiB and more stay with the rows kernel: a lane's offset within an image row has 32 bits (the inputs'
// is below 2 GiB for every problem of this regime, the output's token stride is the caller's).
inline bool small_columns(int gw, int out_token_stride) {
  const int xts = (gw + 15) / 16;
  return 32 * xts <= 3 * gw && (long long)gw * out_token_stride * 2 < (1ll << 32);
}

// Image rows a wave walks down: as many blocks (of kColumnWaves waves) as three a CU, which are resident together, and at least
// four image rows a wave, since two rows of V are read besides.
constexpr int kColumnWaves = 4;
inline int small_column_segment(int units, int gh, int gw, int cus) {
  const int want = std::max(1, (3 * cus + units - 1) / units * kColumnWaves / ((gw + 15) / 16));
  return std::max(std::min(4, gh), (gh + want - 1) / want);
}

// --- many agents (large_broadcast_cols_kernel), with half-resized bias tables ---
constexpr int kColumnRows = 16;          // image rows of a block
constexpr int kMaxColumnParts = 6;       // cell rows of the tables that a block can hold
// Cell rows of the tables a block can need: its image rows are 15 apart at most, and one more for the upper neighbour.  0: the
// kernel does not serve the problem (so many cells that a stage would hold too many of them, e.g. a block grid of half the image's
// rows; up to 64 cells the rounding of a source coordinate crosses no further cell; 32-bit offsets in the row component, the
// other table is below 2 GiB).
inline int large_column_parts(int n, int gh, int cells) {
  if (cells > 64 || (long long)((n + 63) / 64 * 64) * gh * 4 >= (1ll << 31)) return 0;
  const int parts = std::min(cells, (kColumnRows - 1) * cells / gh + 3);
  return parts <= kMaxColumnParts ? parts : 0;
}
// --- many agents, aggregation (large_aggregate_cols_kernel), with half-resized bias tables ---
// A tile is 16 columns x 4 image rows whatever the image: not where more than half as many places again would lie beside it.  Up to 64
// padded channels the kernels in rows run four waves a block up to 256 agents, which is as fast (whole forward, rows / columns in
// us, d = 64: 16 units of 80 x 100 tokens x 256 agents 114 / 119, 96 of 77 x 40 x 81 161 / 166; d = 32 79 / 79, 89 / 92); above, a
// tile should seldom lie across cell rows (d = 64: 4 of 96 x 96 x 576 82 / 76, 24 of 90 x 36 x 360 98 / 94; 3 of 50 x 52 x 400, seven
// image rows a cell row, 58 / 62).  At 128 columns were never slower (192 of 24 x 24 x 144 353 / 252, 4 of 7 x 100 x 90 83 / 72).
// 32-bit offsets: in a head's table and row component, and of a tile's last image row in a unit (which is below 2 GiB) from its
// first.
inline bool large_aggregate_columns(int padded_width, int n, int gh, int gw, int cells) {
  const long long ld = (n + 63) / 64 * 64;
  if (gw % 4 != 0 || gh < 4 || cells * (gw / 4) * ld * 16 >= (1ll << 31) || gh * ld * 4 >= (1ll << 31)) return false;
  const long long tokens = (long long)((gw + 15) / 16 * 16) * ((gh + 3) / 4 * 4);
  if (padded_width <= 64 && (n <= 256 || gh < 10 * cells)) return false;
  return 2 * tokens <= 3ll * gh * gw;
}
inline long long large_column_blocks(int gh, int gw) {
  return (long long)((gw + 15) / 16) * ((gh + kColumnRows - 1) / kColumnRows);
}
// A block is 16 x 16 tokens whatever the image, the rows kernel's any 256 tokens: in a narrow image, or one that reaches a little
// into its last blocks, columns are more blocks, and what counts is how often all CUs are filled.  The rows kernel runs one block
// per CU, columns two where LDS has room for two.  A round of columns against one of rows, from 1150 problems of 64 .. 1024
// agents and 4 .. 128 image columns: the same at 32 padded channels, two fifths at 128; at 64 the same (three quarters above 256
// agents), and a quarter more with two blocks a CU.  Rows / columns in us at d = 64: 128 units of 36 x 80 tokens x 80 agents 119 /
// 127 (1536 / 1920 blocks), 64 of 36 x 28 x 240 30.8 / 47.2 (256 / 384), 192 of 17 x 8 x 91 18.4 / 33.5 (192 / 384); 32 of 67 x 76 x
// 322 107 / 84 (640 / 800), 8 of 88 x 8 x 96 20.4 / 17.2 (24 / 48).  By this rule no problem of 32 or 128 channels measured above
// 1.05 of the rows kernel, of 64 channels 4 of 479 (worst 1.11).
inline bool large_columns_pay(int padded_width, int parts, int n, int units, int gh, int gw, int cus) {
  const long long cols = units * large_column_blocks(gh, gw), rows = units * (((long long)gh * gw + 255) / 256);
  const int stage_bytes = 3 * 128 * padded_width + (1 + parts) * 4096;      // agents and V_A, row component, cell rows
  const bool two = padded_width <= 64 && 4 * stage_bytes <= 160 * 1024 && cols > cus;
  const long long slots = two ? 2 * cus : cus, rounds = (cols + slots - 1) / slots;
  int cost = 20;      // of a round, in twentieths
  if (padded_width == 128) cost = 8;
  if (padded_width == 64) cost = (two ? 25 : 20) * (n > 256 ? 3 : 4) / 4;
  return cost * rounds <= 20 * ((rows + cus - 1) / cus);
}

}  // namespace aa
