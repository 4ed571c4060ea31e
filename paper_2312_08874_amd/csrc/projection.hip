// Linear projections of the module (Sec. 4.2): Y = X W^T + b for 16-bit elements, rows of whole 16-byte pieces.
//
// The library's product wrote Y without the bias and another kernel went over Y again, element by element, and the
// windows of an image were copied to window-major tensors and back around the attention.  Here the bias is the
// accumulators' first value, so that Y is rounded once, and rows of windows are read and written where the attention
// keeps them.  Small widths are bound by memory, for which three or four blocks per CU keep enough loads in flight; large
// ones by the LDS reads of the operands, which a wave's 64 x 64 tile brings level with its products.  Measured, library +
// bias (+ copies of windows) against this kernel: 100352 rows in windows, width 96: q | k | v 49 + 45 + 30 -> 25 us
// (3.1 TB/s), output 28 + 17 + 9 -> 12; 16384 rows, width 512: 45 + 38 -> 40 us (640 TFLOP/s), 15 + 15 -> 17.
#include "kernels.h"
#include "mfma_common.h"

#include <algorithm>

namespace aa {

namespace {

constexpr int kThreads = 256;      // four waves per block
constexpr int kStep = 64;          // channels of X and W in LDS at a time
constexpr int kLst = kStep + 8;    // LDS row stride in elements: 16-byte reads of 16 rows are free of bank conflicts

struct ProjArgs {
  const uint16_t *X, *W, *b;
  uint16_t* Y;
  int M, O, K;
  ProjRows x, y;
  XcdGrid grid;
};

// Where row m (token m % tokens of image m / tokens) lies: a base for the rows from m0 on and this row's offset from it
// (an image has fewer than 2^30 elements, so that the 128 rows of a block and the images around them fit 32 bits).
__device__ __forceinline__ size_t rows_base(const ProjRows& p, int m0) {
  return p.ww == 0 ? (size_t)m0 * p.ld : (size_t)quotient(m0, p.inv_tokens) * p.wyn * p.wxn * p.heads * p.head_elems;
}
__device__ __forceinline__ unsigned row_offset(const ProjRows& p, int m0, int m) {
  if (p.ww == 0) return (unsigned)(m - m0) * (unsigned)p.ld;
  const int b = quotient(m, p.inv_tokens), t = m - b * p.tokens, y = quotient(t, p.inv_line), x = t - y * p.line;
  const int wy = quotient(y, p.inv_wh), wx = quotient(x, p.inv_ww);
  const unsigned window = ((unsigned)(b - quotient(m0, p.inv_tokens)) * p.wyn + wy) * p.wxn + wx;
  return window * (unsigned)p.heads * (unsigned)p.head_elems + (unsigned)(((y - wy * p.wh) * p.ww + (x - wx * p.ww)) * p.d);
}
__device__ __forceinline__ size_t channel_place(const ProjRows& p, int c) {
  if (p.ww == 0) return (size_t)c;
  const int width = p.heads * p.d, part = quotient(c, p.inv_width), in = c - part * width, hd = quotient(in, p.inv_d);
  return part * p.part_elems + (size_t)hd * p.head_elems + (in - hd * p.d);
}

// uniform base, this lane's element offset (below 2^31)
__device__ __forceinline__ u32x4 load16(const uint16_t* base, unsigned at) {
  typedef const __attribute__((address_space(1))) char* bytes;
  return *(const __attribute__((address_space(1))) u32x4*)((bytes)base + (size_t)at * 2);
}

// Block: BM rows of X times BN rows of W, WN waves along W.  A wave's tiles hold 16 outputs x 16 rows of X; two of
// them take every other four outputs, so that a lane holds eight neighbours of a row of Y, one 16-byte store.
// The blocks of the same rows of X are on one XCD (W, at most a few MB, is in every L2).
template <class E, int BM, int BN, int WN>
__global__ __launch_bounds__(kThreads, BM == 128 && BN == 128 ? 3 : 4) void projection_kernel(ProjArgs a) {
  constexpr int WM = 4 / WN, TM = BM / WM / 16, TN = BN / WN / 16;
  constexpr int PX = BM * 8 / kThreads, PW = BN * 8 / kThreads;      // 16-byte pieces per thread and step
  __shared__ __align__(16) uint16_t xs[BM * kLst], ws[BN * kLst];
  int rows, cols;
  if (!a.grid.decode(blockIdx.x, rows, cols)) return;
  const int m0 = rows * BM, o0 = cols * BN;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w / WN, wn = w % WN;
  const int pr = tid >> 3, pc = (tid & 7) * 8;      // this thread's pieces: rows pr + 32 j, channel pc

  // rows past the last are read from the last one: they do not reach Y
  const uint16_t *Xb = a.X + rows_base(a.x, m0), *Wb = a.W + (size_t)o0 * a.K;
  unsigned px[PX], pw[PW];
#pragma unroll
  for (int j = 0; j < PX; ++j) px[j] = row_offset(a.x, m0, min(m0 + pr + 32 * j, a.M - 1));
#pragma unroll
  for (int j = 0; j < PW; ++j) pw[j] = (unsigned)min(pr + 32 * j, a.O - 1 - o0) * (unsigned)a.K;
  u32x4 vx[PX], vw[PW];
  auto fetch = [&](int k0) {      // channels past the last are zeros
    const bool ok = k0 + pc < a.K;
    const int k = ok ? k0 + pc : 0;
    const unsigned xk = (unsigned)channel_place(a.x, k);
#pragma unroll
    for (int j = 0; j < PX; ++j) vx[j] = load16(Xb, px[j] + xk);
#pragma unroll
    for (int j = 0; j < PW; ++j) vw[j] = load16(Wb, pw[j] + (unsigned)k);
    if (!ok) {
#pragma unroll
      for (int j = 0; j < PX; ++j) vx[j] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < PW; ++j) vw[j] = u32x4{0u, 0u, 0u, 0u};
    }
  };
  fetch(0);

  // output of register i of tile t: ob + 32 (t / 2) + 4 (t % 2) + i
  const int ob = o0 + wn * TN * 16 + 8 * g;
  f32x4 acc[TM][TN];
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    f32x4 first = {0.f, 0.f, 0.f, 0.f};
    const int o = ob + 32 * (t / 2) + 4 * (t % 2);
    if (a.b != nullptr && o < a.O) {
      const u32x2 bv = *reinterpret_cast<const u32x2*>(a.b + o);
      float v0, v1, v2, v3;
      Mx<E>::unpack2(bv[0], v0, v1);
      Mx<E>::unpack2(bv[1], v2, v3);
      first = f32x4{v0, v1, v2, v3};
    }
#pragma unroll
    for (int m = 0; m < TM; ++m) acc[m][t] = first;
  }
  // row r of tile t is output 32 (t / 2) + 8 (r / 4) + 4 (t % 2) + r % 4: W goes to LDS in that order
  const int wr = 16 * ((pr >> 2) & 1) + 4 * (pr >> 3) + (pr & 3);
  const uint16_t* wl = ws + (wn * TN * 16 + r) * kLst + 8 * g;
  const uint16_t* xl = xs + (wm * TM * 16 + r) * kLst + 8 * g;
  for (int k0 = 0; k0 < a.K; k0 += kStep) {
    if (k0 > 0) __syncthreads();      // the last step has been read
#pragma unroll
    for (int j = 0; j < PX; ++j) *reinterpret_cast<u32x4*>(xs + (pr + 32 * j) * kLst + pc) = vx[j];
#pragma unroll
    for (int j = 0; j < PW; ++j) *reinterpret_cast<u32x4*>(ws + (wr + 32 * j) * kLst + pc) = vw[j];
    __syncthreads();
    if (k0 + kStep < a.K) fetch(k0 + kStep);
#pragma unroll
    for (int ks = 0; ks < kStep / 32; ++ks) {
      u32x4 xo[TM], wo[TN];
#pragma unroll
      for (int m = 0; m < TM; ++m) xo[m] = *reinterpret_cast<const u32x4*>(xl + 16 * m * kLst + 32 * ks);
#pragma unroll
      for (int t = 0; t < TN; ++t) wo[t] = *reinterpret_cast<const u32x4*>(wl + 16 * t * kLst + 32 * ks);
#pragma unroll
      for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int m = 0; m < TM; ++m) acc[m][t] = Mx<E>::mma(wo[t], xo[m], acc[m][t]);
      __builtin_amdgcn_sched_barrier(0);      // one step's operands at a time: with both the registers spill
    }
  }
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    const int row = m0 + (wm * TM + m) * 16 + r;
    if (row >= a.M) continue;
    uint16_t* py = a.Y + rows_base(a.y, m0) + row_offset(a.y, m0, row);
#pragma unroll
    for (int t = 0; t < TN; t += 2) {
      const int o = ob + 16 * t;
      if (o >= a.O) continue;
      const f32x4 v = acc[m][t], u = acc[m][t + 1];
      *reinterpret_cast<u32x4*>(py + channel_place(a.y, o)) =
          u32x4{Mx<E>::pack2(v[0], v[1]), Mx<E>::pack2(v[2], v[3]), Mx<E>::pack2(u[0], u[1]), Mx<E>::pack2(u[2], u[3])};
    }
  }
}

template <class E, int BM, int BN, int WN>
hipError_t launch(ProjArgs& a, hipStream_t st) {
  a.grid = XcdGrid::make((a.M + BM - 1) / BM, (a.O + BN - 1) / BN);
  projection_kernel<E, BM, BN, WN><<<dim3((unsigned)a.grid.blocks()), dim3(kThreads), 0, st>>>(a);
  return hipGetLastError();
}

template <class E>
hipError_t dispatch(ProjArgs& a, hipStream_t st) {
  // Columns per block: the least padded width, a column of a narrower block priced higher: it takes 8 / 12 (96) or 6 / 8
  // (64) LDS reads per product where 128 takes 8 / 16.
  auto price = [&](int bn, int per_column) { return (long long)((a.O + bn - 1) / bn) * bn * per_column; };
  const long long p128 = price(128, 10), p96 = price(96, 12), p64 = price(64, 13);
  // Rows per block: 64 while blocks of 128 would leave CUs with fewer than two (1 x 196 tokens, width 192: the call 51 ->
  // 21 us with the library's launches gone; 16384 rows, width 320: 12 us as 640 blocks of 64 rows).
  const long long cols = (a.O + 127) / 128, tall = (long long)((a.M + 127) / 128) * cols;
  const bool low = tall < 2 * kComputeUnits;
  if (p128 <= p96 && p128 <= p64) return low ? launch<E, 64, 128, 2>(a, st) : launch<E, 128, 128, 2>(a, st);
  if (p96 <= p64) return low ? launch<E, 64, 96, 1>(a, st) : launch<E, 128, 96, 1>(a, st);
  return low ? launch<E, 64, 64, 2>(a, st) : launch<E, 128, 64, 2>(a, st);
}

}  // namespace

bool ProjRows::windows(const Layout& l, int heads, int d, long long image_tokens, long long rows, size_t part) {
  const unsigned long long width = (unsigned long long)heads * d, lim = 1ull << 32;
  if ((unsigned long long)rows * image_tokens >= lim || 3 * width * width >= lim) return false;      // quotient()
  ww = l.ww, wh = l.wh, line = l.line, wxn = l.wxn, wyn = l.nwin / l.wxn;
  tokens = (int)image_tokens, this->heads = heads, this->d = d;
  head_elems = (size_t)wh * ww * d, part_elems = part;
  inv_tokens = quotient_inverse(tokens), inv_line = quotient_inverse(line), inv_wh = quotient_inverse(wh);
  inv_ww = quotient_inverse(ww), inv_width = quotient_inverse((int)width), inv_d = quotient_inverse(d);
  return true;
}

hipError_t launch_projection(int dtype, int M, int O, int K, const void* X, const ProjRows& x, const void* W, const void* b,
                             void* Y, const ProjRows& y, hipStream_t st) {
  ProjArgs a{(const uint16_t*)X, (const uint16_t*)W, (const uint16_t*)b, (uint16_t*)Y, M, O, K, x, y, XcdGrid{}};
  return dtype == 2 ? dispatch<ElemBF16>(a, st) : dispatch<ElemF16>(a, st);
}

}  // namespace aa
