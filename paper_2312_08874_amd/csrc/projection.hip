// Linear projections of the module (Sec. 4.2): Y = X W^T + b for 16-bit elements, rows of whole 16-byte pieces.
//
// The library's product wrote Y without the bias and another kernel went over Y again, element by element, and the
// windows of an image were copied to window-major tensors and back around the attention.  Here the bias is the
// accumulators' first value, so that Y is rounded once, and rows of windows are read and written where the attention
// keeps them.  What bounds them is the way of the operands to LDS (a product's step waits for loads asked for one step
// before; products, loads and stores alone take 22, 20 and 15 of 42 us at 16384 rows of width 512): direct loads need no
// registers, so that as many blocks as LDS holds share a CU.  Library + bias (+ copies of windows), operands through
// registers (three blocks of 36 KB per CU), direct loads: 100352 rows in windows, width 96: q | k | v 49 + 45 + 30 -> 25 ->
// 19 us (4.1 TB/s), output 28 + 17 + 9 -> 12.6 -> 10.4; 16384 rows, width 512: 45 + 38 -> 43.7 -> 41.7 us (620 TFLOP/s),
// 15 + 15 -> 18.8 -> 15.2.
#include "kernels.h"
#include "mfma_common.h"
#include "split_rules.h"

#include <algorithm>

namespace aa {

namespace {

struct ProjArgs {
  const uint16_t *X, *W, *b;
  uint16_t* Y;
  int M, O, K;
  ProjRows x, y;
  XcdGrid grid;
};

// Where row m (token m % tokens of image m / tokens) lies: a base for the rows from m0 on and this row's offset from it
// (an image has fewer than 2^30 elements, so that the rows of a block and the two images around them, in bytes, fit 32 bits).
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

#define AA_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
// all but the youngest N of this wave's loads have arrived and its LDS reads are done
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
  asm volatile("" ::: "memory");
}

// Block: BM rows of X times BN rows of W, WN waves along W.  A wave's tiles hold 16 outputs x 16 rows of X; two of
// them take every other four outputs, so that a lane holds eight neighbours of a row of Y, one 16-byte store.
// The blocks of the same rows of X are on one XCD (W, at most a few MB, is in every L2).
// Both operands go to LDS by direct loads, KS channels at a time into a ring of NS stages (two or three); piece c of row R lies in slot
// c ^ swz(R), which spreads the 16 rows of an operand read over all banks.
template <class E, int BM, int BN, int NW, int WN, int KS, int NS, int OCC>
__global__ __launch_bounds__(64 * NW, OCC) void projection_kernel(ProjArgs a) {
  constexpr int WM = NW / WN, TM = BM / WM / 16, TN = BN / WN / 16;
  constexpr int PPR = KS / 8, RPL = 64 / PPR;              // 16-byte pieces per row, rows per wave-wide load
  constexpr int LX = BM / (NW * RPL), LW = (BN / RPL + NW - 1) / NW;      // loads per wave and step
  constexpr bool kEven = BN % (NW * RPL) == 0;      // else the last load of W's tile is the first half of the waves' alone
  constexpr int RB = 2 * KS, kStage = (BM + BN) * RB;
  constexpr unsigned kNone = 0xffffffffu;      // past every buffer: the piece is zeros
  static_assert(LX * NW * RPL == BM && (kEven || (LW * NW - NW / 2) * RPL == BN) && TN % 2 == 0, "whole loads");
  extern __shared__ __align__(1024) unsigned char smem[];
  int rows, cols;
  if (!a.grid.decode(blockIdx.x, rows, cols)) return;
  const int m0 = rows * BM, o0 = cols * BN;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w / WN, wn = w % WN;
  auto swz = [](int R) { return PPR == 8 ? (R >> 1) & 7 : (R >> 2) & 3; };

  // output of register i of tile t: ob + 32 (t / 2) + 4 (t % 2) + i
  const int ob = o0 + wn * TN * 16 + 8 * g;
  u32x2 bias[TN];
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    const int o = ob + 32 * (t / 2) + 4 * (t % 2);
    bias[t] = a.b != nullptr && o < a.O ? *reinterpret_cast<const u32x2*>(a.b + o) : u32x2{0u, 0u};
  }
  // this lane's pieces: rows R0 + 4 RPL j of the tile, slot lane % PPR.  Rows past the last are read from the last one: they
  // do not reach Y.  Row 16 t + r of W's tile is output 32 (t / 2) + 8 (r / 4) + 4 (t % 2) + r % 4.
  const int R0 = RPL * w + lane / PPR, pc = 8 * ((lane % PPR) ^ swz(R0));
  const __amdgpu_buffer_rsrc_t Xrs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.X + rows_base(a.x, m0)), 0, (int)0xfffffff0u, 0x00020000);
  const __amdgpu_buffer_rsrc_t Wrs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.W + (size_t)o0 * a.K), 0, (int)0xfffffff0u, 0x00020000);
  unsigned px[LX], pw[LW];
#pragma unroll
  for (int j = 0; j < LX; ++j) px[j] = 2 * row_offset(a.x, m0, min(m0 + R0 + NW * RPL * j, a.M - 1));
#pragma unroll
  for (int j = 0; j < LW; ++j) {
    const int R = R0 + NW * RPL * j, o = 32 * (R >> 5) + 8 * ((R >> 2) & 3) + 4 * ((R >> 4) & 1) + (R & 3);
    pw[j] = 2 * (unsigned)min(o, a.O - 1 - o0) * (unsigned)a.K;
  }
  auto issue = [&](int step) {      // channels past the last are zeros
    const int k = step * KS + pc;
    const bool ok = k < a.K;
    const unsigned xk = 2 * (unsigned)channel_place(a.x, ok ? k : 0), wk = 2 * (unsigned)k;
    unsigned char* st = smem + (step % NS) * kStage + w * 1024;
#pragma unroll
    for (int j = 0; j < LX; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(Xrs, AA_LDS_PTR(st + NW * 1024 * j), 16, (int)(ok ? px[j] + xk : kNone), 0, 0, 0);
#pragma unroll
    for (int j = 0; j < LW; ++j)
      if (kEven || j < LW - 1 || w < NW / 2)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(Wrs, AA_LDS_PTR(st + BM * RB + NW * 1024 * j), 16, (int)(ok ? pw[j] + wk : kNone), 0, 0, 0);
  };
  const int steps = (a.K + KS - 1) / KS;
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < steps) issue(s);

  f32x4 acc[TM][TN];
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    float v0, v1, v2, v3;
    Mx<E>::unpack2(bias[t][0], v0, v1);
    Mx<E>::unpack2(bias[t][1], v2, v3);
#pragma unroll
    for (int m = 0; m < TM; ++m) acc[m][t] = f32x4{v0, v1, v2, v3};
  }
  const int xl = (wm * TM * 16 + r) * RB, wl = BM * RB + (wn * TN * 16 + r) * RB;
  for (int i = 0; i < steps; ++i) {
    // step i has arrived when at most the loads of the step after it are outstanding
    if (NS == 2 || i + 1 == steps) wait_loads<0>();
    else if (kEven || w < NW / 2) wait_loads<LX + LW>();
    else wait_loads<LX + LW - 1>();
    __builtin_amdgcn_s_barrier();      // step i is visible to every wave, and every wave has read step i - 1
    asm volatile("" ::: "memory");
    if (i + NS - 1 < steps) issue(i + NS - 1);      // into the stage of step i - 1
    const unsigned char* st = smem + (i % NS) * kStage;
#pragma unroll
    for (int ks = 0; ks < KS / 32; ++ks) {
      const int at = 16 * ((4 * ks + g) ^ swz(r));
      u32x4 xo[TM], wo[TN];
#pragma unroll
      for (int m = 0; m < TM; ++m) xo[m] = *reinterpret_cast<const u32x4*>(st + xl + 16 * m * RB + at);
#pragma unroll
      for (int t = 0; t < TN; ++t) wo[t] = *reinterpret_cast<const u32x4*>(st + wl + 16 * t * RB + at);
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

template <class E, int BM, int BN, int NW, int WN, int KS, int NS>
hipError_t launch(ProjArgs& a, hipStream_t st) {
  constexpr size_t lds = (size_t)NS * (BM + BN) * 2 * KS;
  constexpr int waves = std::min<int>(4, 160 * 1024 / (int)lds * NW / 4);      // per SIMD, of the blocks that LDS holds
  a.grid = XcdGrid::make((a.M + BM - 1) / BM, (a.O + BN - 1) / BN);
  auto kernel = projection_kernel<E, BM, BN, NW, WN, KS, NS, waves>;
  const hipError_t err = allow_lds(kernel, lds);
  if (err != hipSuccess) return err;
  kernel<<<dim3((unsigned)a.grid.blocks()), dim3(64 * NW), lds, st>>>(a);
  return hipGetLastError();
}

template <class E, int BM, int KS>
hipError_t columns(ProjArgs& a, int outputs, hipStream_t st) {
  if (outputs == 128) return launch<E, BM, 128, 4, 2, KS, 2>(a, st);
  if (outputs == 96) return launch<E, BM, 96, 4, 1, KS, 2>(a, st);
  if constexpr (KS == 32) return launch<E, BM, 64, 4, 2, KS, 2>(a, st);
  return hipErrorInvalidValue;
}

template <class E>
hipError_t dispatch(ProjArgs& a, hipStream_t st) {
  const ProjectionBlocks b = projection_blocks(a.M, a.O, a.K, kComputeUnits);
  if (b.rows == 256) return launch<E, 256, 128, 8, 2, 32, 3>(a, st);
  if (b.step == 32) return b.rows == 64 ? columns<E, 64, 32>(a, b.outputs, st) : columns<E, 128, 32>(a, b.outputs, st);
  return b.rows == 64 ? columns<E, 64, 64>(a, b.outputs, st) : columns<E, 128, 64>(a, b.outputs, st);
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
