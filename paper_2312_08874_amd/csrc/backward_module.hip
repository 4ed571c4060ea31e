// Module terms of the recomputing backward: the agent-bias tables its kernels read, the sums of the bias gradients
// they leave behind, and the depthwise convolution's parameter gradients.  No atomics, every sum in a fixed order.
#include <type_traits>

#include "backward_fused.h"
#include "mfma_common.h"

namespace aa {

namespace {

// ---------------------------------------------------------------------------
// Tables of both bias kinds (BiasTables) in one launch.  A block makes tiles of 64 agents x 16 columns of `run` cell rows
// (T; the column component and the interpolation along x are the same for all of them) or x 16 image rows (R) in LDS: the components are read with the lanes along their contiguous axis (columns or
// rows for B1, agents for B2) and both orders of T are written in pieces of 256 bytes and more.  The last blocks of a
// kind: the image rows' interpolation along y.  Bound by the tables' bytes; with the lanes always along the agents
// B1's components were read, and ta written, a few bytes per line (8 heads, 1024 agents, 128 x 128 tokens: 126 -> 44 us
// for the 117 MB of both kinds; 3 heads, 49 agents, 14 x 14 tokens, where it is the launches: 14 -> 4 us).  run is as large
// as leaves eight blocks a CU: with one cell row a block the divisions and coordinates were most of the arithmetic (the
// first shape 47 -> 34 us).
// ---------------------------------------------------------------------------
struct TableKind {
  BiasArgs b;
  float *ta, *tx, *rows;
  YInfo* yi;
  int kind, cells, run;      // run: cell rows per block
  unsigned tblocks, rblocks, blocks;
};

__device__ __forceinline__ float floored(float v) { return v < kBiasFloor ? kBiasFloor : v; }      // keeps NaN

template <int KIND>
__device__ __forceinline__ void bias_table_block(const TableKind& k, unsigned block, int n, int gh, int gw, int ld,
                                                 float (&tiles)[2][16][68]) {
  float (&tile)[16][68] = tiles[0];
  const BiasArgs& b = k.b;
  const int tid = threadIdx.x, ats = ld / 64, xts = (gw + 15) / 16, yts = (gh + 15) / 16;
  // entry (i, a) of the tile this thread makes in step j: lanes along the components' contiguous axis
  auto place = [&](int j, int& i, int& al) {
    i = KIND == 1 ? tid & 15 : (tid >> 6) + 4 * j;
    al = KIND == 1 ? (tid >> 4) + 16 * j : tid & 63;
  };
  if (block < k.tblocks) {
    const unsigned runs = (unsigned)((k.cells + k.run - 1) / k.run);
    const int at = block % ats, xt = block / ats % xts, c0 = (int)(block / ats / xts % runs) * k.run, hd = block / ats / xts / runs;
    const int c1 = min(c0 + k.run, k.cells);
    float col[4], fx[4], v0[4], v1[4];
    const float *q0[4], *q1[4];      // the block component's entries on both sides, of the cell row in hand
    bool blk[4];
    const size_t cell_step = KIND == 1 ? (size_t)b.w0 : (size_t)b.w0 * n;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int i, al;
      place(j, i, al);
      const int x = 16 * xt + i, a = 64 * at + al;
      col[j] = x >= gw ? kMaskedScore : 0.0f;      // a column past the image weighs nothing
      blk[j] = b.blk && x < gw && a < n;
      if (x < gw && a < n && b.col) col[j] = KIND == 1 ? b.col[((size_t)hd * n + a) * gw + x] : b.col[((size_t)hd * gw + x) * n + a];
      v0[j] = v1[j] = 0.0f;
      if (blk[j]) {
        int x0, x1;
        bilinear_coord(x, gw, b.w0, x0, x1, fx[j]);
        const size_t step = KIND == 1 ? 1 : n;
        const float* q = KIND == 1 ? b.blk + (((size_t)hd * n + a) * b.h0 + c0) * b.w0 : b.blk + ((size_t)hd * b.h0 + c0) * b.w0 * n + a;
        q0[j] = q + x0 * step, q1[j] = q + x1 * step;
        v0[j] = *q0[j], v1[j] = *q1[j];
      }
    }
    const int wp = 16 * xts;
    for (int cell = c0; cell < c1; ++cell) {
      float (&t)[16][68] = tiles[(cell - c0) & 1];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        int i, al;
        place(j, i, al);
        float v = col[j];
        if (blk[j]) {
          const float f0 = floored(v0[j]), f1 = floored(v1[j]);
          v += f0 + (f1 - f0) * fx[j];
        }
        t[i][al] = 16 * xt + i < gw ? floored(v * kLog2e) : v;
      }
      if (cell + 1 < c1) {      // the next cell row's entries are under way while this one's tile goes out
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (blk[j]) q0[j] += cell_step, q1[j] += cell_step, v0[j] = *q0[j], v1[j] = *q1[j];
      }
      __syncthreads();      // two tiles in turn: the one written next was read before this barrier
      const size_t base = ((size_t)hd * k.cells + cell) * ld * wp;
      {
        const int i = tid & 15, a4 = tid >> 4;
        *reinterpret_cast<f32x4*>(k.ta + base + ((size_t)(16 * at + a4) * wp + 16 * xt + i) * 4) =
            *reinterpret_cast<const f32x4*>(&t[i][4 * a4]);
      }
      const int x4 = tid >> 6, al = tid & 63;
      *reinterpret_cast<f32x4*>(k.tx + base + ((size_t)(4 * xt + x4) * ld + 64 * at + al) * 4) =
          f32x4{t[4 * x4][al], t[4 * x4 + 1][al], t[4 * x4 + 2][al], t[4 * x4 + 3][al]};
    }
  } else if (block < k.tblocks + k.rblocks) {
    block -= k.tblocks;
    const int at = block % ats, yt = block / ats % yts, hd = block / ats / yts;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int i, al;
      place(j, i, al);
      const int y = 16 * yt + i, a = 64 * at + al;
      float v = 0.0f;
      if (y < gh && a < n) v = floored(kLog2e * (KIND == 1 ? b.row[((size_t)hd * n + a) * gh + y] : b.row[((size_t)hd * gh + y) * n + a]));
      tile[i][al] = v;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = (tid >> 6) + 4 * j, al = tid & 63, y = 16 * yt + i;
      if (y < gh) k.rows[((size_t)hd * gh + y) * ld + 64 * at + al] = tile[i][al];
    }
  } else {
    const int y = (int)(block - k.tblocks - k.rblocks) * 256 + tid;
    if (y >= gh) return;
    int i0, i1;
    float f;
    bilinear_coord(y, gh, k.cells, i0, i1, f);
    int next = y + 1;
    for (; next < gh; ++next) {
      int c;
      float g;
      bilinear_coord(next, gh, k.cells, c, i1, g);
      if (c != i0) break;
    }
    k.yi[y] = YInfo{i0, next, i0 >= k.cells - 1 ? 0.0f : f, 0};
  }
}

__global__ __launch_bounds__(256) void bias_tables_kernel(TableKind first, TableKind second, int n, int gh, int gw, int ld,
                                                          int* flags, int n_flags) {
  __shared__ __align__(16) float tile[2][16][68];
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n_flags; i += gridDim.x * 256) flags[i] = 0;
  const bool one = blockIdx.x < first.blocks;
  const unsigned block = one ? blockIdx.x : blockIdx.x - first.blocks;
  const TableKind& k = one ? first : second;
  if (k.kind == 1) bias_table_block<1>(k, block, n, gh, gw, ld, tile);
  else bias_table_block<2>(k, block, n, gh, gw, ld, tile);
}

// cell rows [c0, c1] that the image rows of segment s touch
__device__ __forceinline__ void segment_cells(int s, int seg_len, int gh, int cells, int& c0, int& c1) {
  int up;
  float f;
  bilinear_coord(s * seg_len, gh, cells, c0, up, f);
  bilinear_coord(min(gh, (s + 1) * seg_len) - 1, gh, cells, c1, up, f);
  c1 = min(c1 + 1, cells - 1);
}

// What the gradients of one bias kind are made from and where they go (null: not wanted)
struct GradKind {
  const f32x4 *gt, *sum;      // sum: of the parts, = gt where there is a single one
  f32x4* total;               // where the sum goes (null: a single part)
  const float* gr;
  float *col, *row, *blk;
  int kind, segs, seg_len, cells, w0;
  float live;                 // 0: the softmax has a single entry, is constant, and its scores' gradients are zero (the
                              // parts hold the rounding error of a difference of equal terms)
  unsigned sblocks, cblocks, rblocks, blocks;
};

// sum [heads][cells][wp / 4][ld] of four columns each: the parts of the batch's units and their segments, in order
__global__ __launch_bounds__(256) void bias_grad_sum_kernel(GradKind first, GradKind second, int batch, int heads, int gh,
                                                            size_t per_cell) {
  const bool one = blockIdx.x < first.sblocks;
  const GradKind& k = one ? first : second;
  const size_t i = (size_t)(one ? blockIdx.x : blockIdx.x - first.sblocks) * 256 + threadIdx.x;
  if (i >= (size_t)heads * k.cells * per_cell) return;
  const size_t e = i % per_cell;
  const int cell = (int)(i / per_cell % k.cells), hd = (int)(i / per_cell / k.cells);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < k.segs; ++s) {
    int c0, c1;
    segment_cells(s, k.seg_len, gh, k.cells, c0, c1);
    if (cell < c0 || cell > c1) continue;
    const f32x4* p = k.gt + (((size_t)hd * k.segs + s) * k.cells + cell) * per_cell + e;
    const size_t step = (size_t)heads * k.segs * k.cells * per_cell;
#pragma unroll 16      // a round trip to memory per sixteen images, not per four
    for (int bt = 0; bt < batch; ++bt) acc += p[bt * step];
  }
  k.total[i] = acc;
}

// The same for a batch of eight images and more: the four waves of a block share out the images of 64 sums, each in order and
// eight of them asked for at once, and are added in order.  (One thread over the batch is a chain of round trips to memory
// with too few threads to hide them: 3 heads, 64 images, 49 agents, 14 x 14 tokens 9.4 -> 5.6 us, 6 heads, 8 images, 63 agents, 31 x 43
// tokens 11 -> 6.6 us.)
__global__ __launch_bounds__(256) void bias_grad_batch_sum_kernel(GradKind first, GradKind second, int batch, int heads, int gh,
                                                                  unsigned per_cell) {
  __shared__ f32x4 red[4][64];
  const bool one = blockIdx.x < first.sblocks;
  const GradKind& k = one ? first : second;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned i = (one ? blockIdx.x : blockIdx.x - first.sblocks) * 64u + lane;
  const unsigned last = (unsigned)heads * k.cells * per_cell - 1, at = min(i, last);
  const unsigned hc = at / per_cell, e = at - hc * per_cell, hd = hc / k.cells;
  const int cell = (int)(hc - hd * k.cells), b0 = (w * batch) >> 2, b1 = ((w + 1) * batch) >> 2;
  const size_t step = (size_t)heads * k.segs * k.cells * per_cell;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < k.segs; ++s) {
    int c0, c1;
    segment_cells(s, k.seg_len, gh, k.cells, c0, c1);
    if (cell < c0 || cell > c1) continue;
    const f32x4* p = k.gt + (((size_t)hd * k.segs + s) * k.cells + cell) * per_cell + e;
    int b = b0;
    for (; b + 8 <= b1; b += 8) {
      f32x4 v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = p[(b + j) * step];
#pragma unroll
      for (int j = 0; j < 8; ++j) acc += v[j];
    }
    for (; b + 2 <= b1; b += 2) {
      const f32x4 v0 = p[b * step], v1 = p[(b + 1) * step];
      acc += v0;
      acc += v1;
    }
    if (b < b1) acc += p[b * step];
  }
  red[w][lane] = acc;
  __syncthreads();
  if (w == 0 && i <= last) k.total[i] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// The components' gradients from the sums: column blocks (a thread has an agent and four columns), then row blocks (a
// block has 64 agents and four image rows, its waves share out the parts), then block-cell blocks (one output element
// per thread, over the columns that can touch it), lanes along the agents; after both kinds the convolution's
// parameter gradients from their slices.  One launch, because small problems are a chain of launches (3 heads, batch
// 64, 49 agents, 14 x 14 tokens: 81 -> 14 us with the sums above); there a thread walking the batch alone took a round
// trip per image.  8 heads, 1024 agents, 128 x 128 tokens: 123 -> 71 us, bound by reading the parts and sums (150 MB).
template <int KIND>
__device__ __forceinline__ void bias_grad_block(const GradKind& k, unsigned block, int batch, int heads, int n, int gh, int gw,
                                                int ld, float (&red)[4][4][64]) {
  const int xts = (gw + 15) / 16, wp = 16 * xts, tid = threadIdx.x;
  const size_t per_cell = (size_t)wp / 4 * ld;
  if (block < k.cblocks) {
    const int gw4 = (gw + 3) / 4;
    const size_t i = (size_t)block * 256 + tid;
    const int a = (int)(i % n), x4 = (int)(i / n % gw4), hd = (int)(i / n / gw4);
    if (hd >= heads) return;
    const f32x4* p = k.sum + (size_t)hd * k.cells * per_cell + (size_t)x4 * ld + a;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int c = 0; c < k.cells; ++c) v += p[c * per_cell];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int x = 4 * x4 + j;
      if (x < gw) k.col[KIND == 1 ? ((size_t)hd * n + a) * gw + x : ((size_t)hd * gw + x) * n + a] = k.live * v[j];
    }
  } else if (block < k.cblocks + k.rblocks) {
    block -= k.cblocks;
    const int ats = (n + 63) / 64, gh4 = (gh + 3) / 4;
    const int at = block % ats, y0 = 4 * (int)(block / ats % gh4), hd = block / ats / gh4;
    const int lane = tid & 63, w = tid >> 6;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    const size_t part = (size_t)gh * ld;
    const float* p = k.gr + (size_t)hd * xts * part + 64 * at + lane;      // ld reaches past the last tile's agents
#pragma unroll 4
    for (int q = w; q < batch * xts; q += 4) {
      const int bt = q / xts, t = q - bt * xts;
      const float* r = p + ((size_t)bt * heads * xts + t) * part;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] += r[(size_t)min(y0 + j, gh - 1) * ld];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) red[w][j][lane] = v[j];
    __syncthreads();
    const int j = KIND == 1 ? tid & 3 : w, al = KIND == 1 ? tid >> 2 : lane, a = 64 * at + al, y = y0 + j;
    if (a < n && y < gh)
      k.row[KIND == 1 ? ((size_t)hd * n + a) * gh + y : ((size_t)hd * gh + y) * n + a] =
          k.live * ((red[0][j][al] + red[1][j][al]) + (red[2][j][al] + red[3][j][al]));
  } else {
    const size_t i = (size_t)(block - k.cblocks - k.rblocks) * 256 + tid;
    const int a = (int)(i % n), q = (int)(i / n % k.w0), cell = (int)(i / n / k.w0 % k.cells), hd = (int)(i / n / k.w0 / k.cells);
    if (hd >= heads) return;
    // columns whose source coordinate lies within one cell of q, with a column to spare on both sides (the weights
    // decide); the first and the last cell also take what the clamping sends there
    const float scale = (float)gw / (float)k.w0;
    const int lo = q == 0 ? 0 : max((int)(((float)q - 0.5f) * scale - 1.5f), 0);
    const int hi = q == k.w0 - 1 ? gw : min((int)(((float)q + 1.5f) * scale + 1.5f), gw);
    const f32x4* p = k.sum + ((size_t)hd * k.cells + cell) * per_cell + a;
    float v = 0.0f;
#pragma unroll 4
    for (int x4 = lo / 4; 4 * x4 < hi; ++x4) {
      const f32x4 s = p[(size_t)x4 * ld];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        int x0, x1;
        float fx;
        bilinear_coord(min(4 * x4 + j, gw - 1), gw, k.w0, x0, x1, fx);
        const float wx = 4 * x4 + j < gw ? (x0 == q ? 1.0f - fx : 0.0f) + (x1 == q ? fx : 0.0f) : 0.0f;
        if (wx != 0.0f) v = fmaf(wx, s[j], v);
      }
    }
    const size_t cellq = (size_t)cell * k.w0 + q;
    k.blk[KIND == 1 ? ((size_t)hd * n + a) * k.cells * k.w0 + cellq : ((size_t)hd * k.cells * k.w0 + cellq) * n + a] = k.live * v;
  }
}

struct DwcTotal {
  const float* part;
  float *dw, *db;         // either may be null
  int slices, count;      // count: heads * d
};

__global__ __launch_bounds__(256) void param_grad_out_kernel(GradKind first, GradKind second, DwcTotal dwc, int batch, int heads,
                                                             int n, int d, int gh, int gw, int ld) {
  __shared__ float red[4][4][64];
  unsigned block = blockIdx.x;
  if (block < first.blocks + second.blocks) {
    const bool one = block < first.blocks;
    const GradKind& k = one ? first : second;
    if (!one) block -= first.blocks;
    if (k.kind == 1) bias_grad_block<1>(k, block, batch, heads, n, gh, gw, ld, red);
    else bias_grad_block<2>(k, block, batch, heads, n, gh, gw, ld, red);
    return;
  }
  // one wave per (head, channel): lane l adds the slices l, l + 64, ... in order, the lanes are added by a fixed tree
  block -= first.blocks + second.blocks;
  const int hc = (int)block * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (hc >= dwc.count) return;
  const int hd = hc / d, c = hc - hd * d;
  float acc[10];
#pragma unroll
  for (int k = 0; k < 10; ++k) acc[k] = 0.0f;
  for (int s = lane; s < dwc.slices; s += 64) {
    const float* q = dwc.part + (((size_t)hd * dwc.slices + s) * d + c) * 10;
#pragma unroll
    for (int k = 0; k < 10; ++k) acc[k] += q[k];
  }
#pragma unroll
  for (int k = 0; k < 10; ++k) acc[k] = wave_sum(acc[k]);
  if (lane == 0) {
    if (dwc.dw) {
#pragma unroll
      for (int k = 0; k < 9; ++k) dwc.dw[(size_t)hc * 9 + k] = acc[k];
    }
    if (dwc.db) dwc.db[hc] = acc[9];
  }
}

// ---------------------------------------------------------------------------
// DWC parameter gradients: dw[c][tap] = sum over batch and tokens of dO[y,x,c] V[y + p, x + q, c], db[c] = sum dO.
// A thread owns a 16-byte piece of the channels of an image column and walks down V's rows with three rows of dO in
// registers, so that a row costs three 16-byte reads of V (two of them shared with the neighbouring columns through
// L1) and one of dO, asked for three rows ahead (read where it was used, a row cost a round trip to memory); CHP = 16-byte
// pieces per token rounded up to a power of two.  The lanes of a block are added by a fixed tree of register permutations
// (through LDS they took as long as ten rows), the blocks by param_grad_out_kernel.  96 units of 3136 tokens, d = 32: 28 ->
// 19 us.
// A block: a head and a slice of 256 / CHP (column, row segment, image) items.
// ---------------------------------------------------------------------------
template <class E>
struct Piece {      // 16 bytes of elements as floats
  using S = uint16_t;
  static constexpr int kCount = 8;
  static __device__ __forceinline__ void unpack(u32x4 p, float* o) {
#pragma unroll
    for (int i = 0; i < 4; ++i) Mx<E>::unpack2(p[i], o[2 * i], o[2 * i + 1]);
  }
};
template <>
struct Piece<ElemF32> {
  using S = float;
  static constexpr int kCount = 4;
  static __device__ __forceinline__ void unpack(u32x4 p, float* o) {
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = __uint_as_float(p[i]);
  }
};

// sum of v over the lanes with the same lane % CHP, in each of them
template <int CHP>
__device__ __forceinline__ float lane_sum(float v) {
  auto rotated = [](float x, auto by) {      // within 16 lanes
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + decltype(by)::value, 0xF, 0xF, false));
  };
  if constexpr (CHP <= 8) v += rotated(v, std::integral_constant<int, 8>{});
  if constexpr (CHP <= 4) v += rotated(v, std::integral_constant<int, 4>{});
  if constexpr (CHP <= 2) v += rotated(v, std::integral_constant<int, 2>{});
  if constexpr (CHP <= 16) return xor16_32_sum(v);
  const uint32_t b = __float_as_uint(v);
  const auto h = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

template <class E, int CHP>
__global__ __launch_bounds__(256, 2) void dwc_param_kernel(const typename Piece<E>::S* __restrict__ V,
                                                        const typename Piece<E>::S* __restrict__ dO,
                                                        float* __restrict__ part, int heads, int d, Layout lay, int gh, int gw,
                                                        int segs, int seg_len, int items, int slices, XcdGrid xg) {
  using S = typename Piece<E>::S;
  constexpr int P = Piece<E>::kCount;
  __shared__ float red[4][CHP][10 * P];
  int slice, hd;      // the heads of a slice share the lines of token-major rows (see XcdGrid)
  if (!xg.decode(blockIdx.x, slice, hd)) return;      // before the barrier
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int ch = tid % CHP;
  const int item = slice * (256 / CHP) + tid / CHP;
  float acc[10][P];
#pragma unroll
  for (int k = 0; k < 10; ++k)
#pragma unroll
    for (int i = 0; i < P; ++i) acc[k][i] = 0.0f;
  if (item < items && ch * P < d) {
    const int x = item % gw, s = item / gw % segs, b = item / gw / segs;
    const int u = b * heads + hd, pitch = lay.pitch(gw);
    const S* v = V + lay.in_unit(u, heads) + ch * P;
    const S* g = dO + lay.out_unit(u, heads) + ch * P + (size_t)x * lay.on;
    const int y0 = s * seg_len, y1 = min(gh, y0 + seg_len);
    // addresses are clamped into the image: what a column beside it adds is struck from the sums at the end, rows of dO above
    // and below it are passed over (not multiplied as zeros: V may hold infinities)
    const S* vx[3] = {v + (size_t)max(x - 1, 0) * lay.sn, v + (size_t)x * lay.sn, v + (size_t)min(x + 1, gw - 1) * lay.sn};
    const size_t vrow = (size_t)pitch * lay.sn, grow = (size_t)pitch * lay.on;
    struct Row {
      u32x4 v[3], g;      // row y of V, row y + 1 of dO
    } r0, r1, r2;
    auto load_g = [&](int y) { return *reinterpret_cast<const u32x4*>(g + (size_t)min(max(y, 0), gh - 1) * grow); };
    auto load = [&](int y, Row& r) {
      const size_t at = (size_t)min(y, gh - 1) * vrow;
#pragma unroll
      for (int q = 0; q < 3; ++q) r.v[q] = *reinterpret_cast<const u32x4*>(vx[q] + at);
      r.g = load_g(y + 1);
    };
    float win[3][P];      // rows y - 1, y, y + 1 of dO (rotating)
    auto row = [&](int y, Row& r, const float (&above)[P], const float (&here)[P], float (&below)[P]) {
      float v[3][P];
      Piece<E>::unpack(r.g, below);
#pragma unroll
      for (int q = 0; q < 3; ++q) Piece<E>::unpack(r.v[q], v[q]);
      load(y + 3, r);
#pragma unroll
      for (int i = 0; i < P; ++i) acc[9][i] += here[i];
      auto taps = [&](int first, const float (&o)[P]) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
          for (int i = 0; i < P; ++i) acc[first + q][i] = fmaf(o[i], v[q][i], acc[first + q][i]);
      };
      taps(3, here);
      if (y + 1 < gh) taps(0, below);
      if (y > 0) taps(6, above);
    };
    const u32x4 g0 = load_g(y0 - 1), g1 = load_g(y0);
    load(y0, r0);
    load(y0 + 1, r1);
    load(y0 + 2, r2);
    Piece<E>::unpack(g0, win[0]);
    Piece<E>::unpack(g1, win[1]);
    int y = y0;
    for (; y + 3 <= y1; y += 3) {
      row(y, r0, win[0], win[1], win[2]);
      row(y + 1, r1, win[1], win[2], win[0]);
      row(y + 2, r2, win[2], win[0], win[1]);
    }
    if (y < y1) row(y, r0, win[0], win[1], win[2]);
    if (y + 1 < y1) row(y + 1, r1, win[1], win[2], win[0]);
#pragma unroll
    for (int k = 0; k < 9; k += 3)
#pragma unroll
      for (int i = 0; i < P; ++i) {
        if (x == 0) acc[k][i] = 0.0f;
        if (x == gw - 1) acc[k + 2][i] = 0.0f;
      }
  }
#pragma unroll
  for (int k = 0; k < 10; ++k)
#pragma unroll
    for (int i = 0; i < P; ++i) acc[k][i] = lane_sum<CHP>(acc[k][i]);
  if (lane < CHP)
#pragma unroll
    for (int k = 0; k < 10; ++k)
#pragma unroll
      for (int i = 0; i < P; ++i) red[w][lane][i * 10 + k] = acc[k][i];
  __syncthreads();
  for (int i = tid; i < d * 10; i += 256)      // channel-major, ten sums each
    part[((size_t)hd * slices + slice) * d * 10 + i] =
        (red[0][i / (10 * P)][i % (10 * P)] + red[1][i / (10 * P)][i % (10 * P)]) + (red[2][i / (10 * P)][i % (10 * P)] + red[3][i / (10 * P)][i % (10 * P)]);
}

// 16-byte pieces per token, rounded up to a power of two, and the row segments an image column is cut into: as many as
// give about 512 blocks, of at least four rows (a segment reads two rows of V it does not own)
struct DwcPlan {
  int chp, segs, seg_len, items, slices;
};
DwcPlan dwc_plan(const Problem& p) {
  DwcPlan q{};
  const int pieces = p.d / (p.dtype == 0 ? 4 : 8);
  q.chp = pieces <= 2 ? 2 : (pieces <= 4 ? 4 : (pieces <= 8 ? 8 : (pieces <= 16 ? 16 : 32)));
  const int batch = p.units / p.heads, per_block = 256 / q.chp;
  const long long cols = (long long)batch * p.gw;
  const long long blocks = (cols + per_block - 1) / per_block * p.heads;
  long long segs = (512 + blocks - 1) / blocks;
  segs = std::max<long long>(1, std::min<long long>(segs, p.gh / 4));
  q.seg_len = (int)((p.gh + segs - 1) / segs);
  q.segs = (p.gh + q.seg_len - 1) / q.seg_len;
  q.items = (int)(cols * q.segs);
  q.slices = (q.items + per_block - 1) / per_block;
  return q;
}

}  // namespace

hipError_t launch_backward_bias_tables(const Problem& p, const BiasTables (&t)[2], const bool (&used)[2], int* flags, int n_flags,
                                       hipStream_t st) {
  TableKind kinds[2] = {};
  int ld = 0;
  for (int i = 0; i < 2; ++i) {
    if (!used[i]) continue;
    TableKind& k = kinds[i];
    k.kind = i == 0 ? 2 : 1, k.b = i == 0 ? p.b2 : p.b1, k.cells = t[i].cells, ld = t[i].ld;
    k.ta = const_cast<float*>(t[i].ta), k.tx = const_cast<float*>(t[i].tx), k.rows = const_cast<float*>(t[i].rows);
    k.yi = const_cast<YInfo*>(t[i].yi);
    const size_t ats = (size_t)p.heads * (ld / 64);
    const size_t columns = ats * ((p.gw + 15) / 16);
    k.run = (int)std::max<size_t>(1, std::min<size_t>(k.cells, columns * k.cells / (4 * kComputeUnits)));
    k.tblocks = (unsigned)(columns * ((k.cells + k.run - 1) / k.run));
    k.rblocks = k.rows ? (unsigned)(ats * ((p.gh + 15) / 16)) : 0;
    k.blocks = k.tblocks + k.rblocks + (unsigned)((p.gh + 255) / 256);
  }
  const unsigned blocks = kinds[0].blocks + kinds[1].blocks;
  if (blocks == 0) return hipSuccess;
  bias_tables_kernel<<<dim3(blocks), dim3(256), 0, st>>>(kinds[0], kinds[1], p.n, p.gh, p.gw, ld, flags, n_flags);
  return hipGetLastError();
}

size_t dwc_param_part_floats(const Problem& p) { return (size_t)p.heads * dwc_plan(p).slices * p.d * 10; }

hipError_t launch_backward_param_grads(const Problem& p, const BiasGradParts (&parts)[2], const BackwardParamGrads& pg,
                                       const void* V, const void* dO, float* dwc_part, hipStream_t st) {
  const int batch = p.units / p.heads, wp = (p.gw + 15) / 16 * 16;
  GradKind kinds[2] = {};
  int ld = 64;
  for (int i = 0; i < 2; ++i) {
    const BiasGradParts& q = parts[i];
    GradKind& k = kinds[i];
    k.kind = i == 0 ? 2 : 1;
    if (!q.gt) continue;
    ld = q.ld;
    k.col = i == 0 ? pg.db2_col : pg.db1_col, k.row = i == 0 ? pg.db2_row : pg.db1_row, k.blk = i == 0 ? pg.db2_blk : pg.db1_blk;
    k.gt = k.sum = reinterpret_cast<const f32x4*>(q.gt), k.gr = q.gr;
    k.segs = q.segs, k.seg_len = q.seg_len, k.cells = q.cells, k.w0 = pg.w0;
    k.live = (k.kind == 1 ? p.N : p.n) > 1 ? 1.0f : 0.0f;
    // a single part is the sum itself, where the image rows touch every cell row (at least as many rows as cells)
    if ((k.col || k.blk) && (batch > 1 || q.segs > 1 || q.cells > p.gh)) {
      k.sum = k.total = reinterpret_cast<f32x4*>(q.sum);
      const size_t per_block = batch >= 8 ? 64 : 256;
      k.sblocks = (unsigned)(((size_t)p.heads * q.cells * (wp / 4) * ld + per_block - 1) / per_block);
    }
    k.cblocks = k.col ? (unsigned)(((size_t)p.heads * ((p.gw + 3) / 4) * p.n + 255) / 256) : 0;
    k.rblocks = k.row ? (unsigned)((size_t)p.heads * ((p.gh + 3) / 4) * ((p.n + 63) / 64)) : 0;
    k.blocks = k.cblocks + k.rblocks + (k.blk ? (unsigned)(((size_t)p.heads * pg.h0 * pg.w0 * p.n + 255) / 256) : 0);
  }
  if (const unsigned blocks = kinds[0].sblocks + kinds[1].sblocks) {
    const size_t per_cell = (size_t)(wp / 4) * ld;
    if (batch >= 8)
      bias_grad_batch_sum_kernel<<<dim3(blocks), dim3(256), 0, st>>>(kinds[0], kinds[1], batch, p.heads, p.gh, (unsigned)per_cell);
    else
      bias_grad_sum_kernel<<<dim3(blocks), dim3(256), 0, st>>>(kinds[0], kinds[1], batch, p.heads, p.gh, per_cell);
  }
  DwcTotal total{};
  if (p.dwc_w && (pg.ddwc_w || pg.ddwc_b)) {
    const DwcPlan q = dwc_plan(p);
    const XcdGrid xg = XcdGrid::make(q.slices, p.heads);
    const dim3 grid((unsigned)xg.blocks());
    auto go = [&](auto kernel, auto elem) {
      using S = typename Piece<decltype(elem)>::S;
      kernel<<<grid, dim3(256), 0, st>>>((const S*)V, (const S*)dO, dwc_part, p.heads, p.d, p.lay, p.gh, p.gw, q.segs, q.seg_len,
                                         q.items, q.slices, xg);
    };
    auto by_pieces = [&](auto elem) {
      using E = decltype(elem);
      switch (q.chp) {
        case 2: go(dwc_param_kernel<E, 2>, elem); break;
        case 4: go(dwc_param_kernel<E, 4>, elem); break;
        case 8: go(dwc_param_kernel<E, 8>, elem); break;
        case 16: go(dwc_param_kernel<E, 16>, elem); break;
        default: go(dwc_param_kernel<E, 32>, elem); break;      // fp32 only
      }
    };
    if (p.dtype == 2) by_pieces(ElemBF16{});
    else if (p.dtype == 1) by_pieces(ElemF16{});
    else by_pieces(ElemF32{});
    total = DwcTotal{dwc_part, pg.ddwc_w, pg.ddwc_b, q.slices, p.heads * p.d};
  }
  const unsigned blocks = kinds[0].blocks + kinds[1].blocks + (unsigned)((total.count + 3) / 4);
  if (blocks == 0) return hipGetLastError();
  param_grad_out_kernel<<<dim3(blocks), dim3(256), 0, st>>>(kinds[0], kinds[1], total, batch, p.heads, p.n, p.d, p.gh, p.gw, ld);
  return hipGetLastError();
}

}  // namespace aa
