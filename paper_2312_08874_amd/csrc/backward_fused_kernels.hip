// Recomputing backward (backward_fused.inc): the kernels without an agent bias, the sums over the token ranges and the
// host side.
#include "backward_fused.inc"

#include <algorithm>

namespace aa {

// compiled by backward_bias_{bf16,f16}.hip and backward_f32.hip
#define AA_EXTERN(E, BIAS)                                                                                       \
  extern template hipError_t launch_token<E, BIAS>(int, int, int, const TokenArgs&, dim3, size_t, hipStream_t);   \
  extern template hipError_t launch_agent<E, BIAS>(int, int, int, const AgentArgs&, dim3, size_t, hipStream_t);   \
  extern template hipError_t launch_both<E, BIAS>(int, int, const AgentArgs&, dim3, size_t, hipStream_t);
AA_EXTERN(ElemBF16, true)
AA_EXTERN(ElemF16, true)
AA_EXTERN(ElemF32, false)
AA_EXTERN(ElemF32, true)
#undef AA_EXTERN

namespace {

// ---------------------------------------------------------------------------
// Sums over the token ranges, in order.  Rows are the agents of all units; lpr lanes (a power of two, at least d / 4) take a
// row, four channels a lane.  What bounds them is the way to memory: the ranges are asked for eight at a time, so that a row
// costs a trip or two instead of one per range, and a block takes 8 to 32 rows (one 64-lane block per row and a trip per
// range before: merge of 192 units x 49 rows of 64 channels in two ranges 7.6 -> 4.2 us, of 8 x 1024 in four 7.4 -> 5.3).
// ---------------------------------------------------------------------------
struct SumRows {
  int rows, n, d, S, lpr_log2;
  __device__ __forceinline__ bool place(int& row, int& c, size_t& first) const {      // first: of range 0, in rows
    row = blockIdx.x * (kThreads >> lpr_log2) + (threadIdx.x >> lpr_log2);
    c = 4 * (threadIdx.x & ((1 << lpr_log2) - 1));
    const int there = min(row, rows - 1), u = unit(there);
    first = (size_t)u * S * n + (there - u * n);
    return row < rows && c < d;
  }
  __device__ __forceinline__ int unit(int r) const { return (int)((unsigned)r / (unsigned)n); }
  // sum over a row's lanes
  __device__ __forceinline__ float row_sum(float v) const {
    for (int m = 1; m < 1 << lpr_log2; m <<= 1) v += __shfl_xor(v, m);
    return v;
  }
};
__device__ __forceinline__ f32x4 row4(const float* p, size_t row, int d, int c) { return load_global<f32x4>(p + row * d + c); }

constexpr int kMaxRanges = 64;      // of a unit's tokens

// log-sum-exp merge of the recomputed aggregation: V_A (fp32 and element type), reference and weight of the rows (log2
// domain; w1 null: the log-sum-exp, no weight)
template <class E>
__global__ __launch_bounds__(kThreads) void fused_merge_kernel(SumRows g, const float* acc, const float* pm, const float* pl,
                                                               float* VAf, typename E::T* VAe, float* lse1, float* w1, int* large) {
  using X = El<E>;
  int row, c;
  size_t first;
  const bool ok = g.place(row, c, first);
  // the rows of eight ranges and their references and weights are asked for together; the references of later ranges before
  float M = -INFINITY, m[8], l[8];
  f32x4 v = {0.f, 0.f, 0.f, 0.f}, x[8];
  float L = 0.f;
  constexpr float kShare = 1.0f / kMaxRanges;      // (a power of two) what fits fp32 in every range fits it in their sum
  auto fetch = [&](int s0) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const size_t at = first + (size_t)min(s0 + k, g.S - 1) * g.n;
      m[k] = load_global<float>(pm + at), l[k] = load_global<float>(pl + at);
      x[k] = row4(acc, at, g.d, c < g.d ? c : 0);
    }
  };
  fetch(0);
  for (int s0 = 8; s0 < g.S; s0 += 8) {
    float later[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) later[k] = load_global<float>(pm + first + (size_t)min(s0 + k, g.S - 1) * g.n);
#pragma unroll
    for (int k = 0; k < 8; ++k) M = fmaxf(M, later[k]);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) M = fmaxf(M, m[k]);
  for (int s0 = 0;;) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (s0 + k >= g.S) continue;      // (not a weight of 0: a row may hold infinities)
      const float w = fast_exp2(m[k] - M);
      L = fmaf(l[k], w, L);
      v += x[k] * (w * kShare);
    }
    if ((s0 += 8) >= g.S) break;
    fetch(s0);
  }
  if (!ok) return;
  v *= (1.0f / L) * (1.0f / kShare);
  const size_t o = (size_t)row * g.d + c;
  *reinterpret_cast<f32x4*>(VAf + o) = v;
  if constexpr (X::kBytes == 2) *reinterpret_cast<typename X::P4*>(VAe + o) = X::pack4(v[0], v[1], v[2], v[3]);      // fp32: the same array
  if (c == 0) {
    const bool apart = w1 && (X::kBytes == 4 || fabsf(M) > kLargeRef);
    lse1[row] = apart ? M : M + __builtin_amdgcn_logf(L);
    if (w1) w1[row] = apart ? 1.0f / L : 1.0f;
    if (large && apart) set_flag(large + g.unit(row));
  }
}

// dV_A = sum of the ranges (element type), D1 = rowsum(dV_A o V_A), dA = c2 * sum of the ranges
template <class E>
__global__ __launch_bounds__(kThreads) void fused_reduce_bc_kernel(SumRows g, const float* pva, const float* pa, const float* VAf,
                                                                   typename E::T* dVAe, float* D1, float* dAf, float c2) {
  using X = El<E>;
  int row, c;
  size_t first;
  const bool ok = g.place(row, c, first);
  f32x4 v = {0.f, 0.f, 0.f, 0.f}, q = v;
  for (int s0 = 0; s0 < g.S; s0 += 8) {
    f32x4 x[8], y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const size_t at = first + (size_t)min(s0 + k, g.S - 1) * g.n;
      x[k] = row4(pva, at, g.d, c < g.d ? c : 0), y[k] = row4(pa, at, g.d, c < g.d ? c : 0);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (s0 + k < g.S) v += x[k], q += y[k];
  }
  float dot = 0.f;
  const size_t o = (size_t)row * g.d + c;
  if (ok) {
    const typename X::P4 e = X::pack4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<typename X::P4*>(dVAe + o) = e;
    *reinterpret_cast<f32x4*>(dAf + o) = q * c2;
    const f32x4 p = X::unpack4(e) * load_global<f32x4>(VAf + o);
    dot = (p[0] + p[1]) + (p[2] + p[3]);
  }
  dot = g.row_sum(dot);
  if (ok && c == 0) D1[row] = dot;
}

// dA += c1 * sum of the ranges; written in the element type too when the agents were handed in
template <class E>
__global__ __launch_bounds__(kThreads) void fused_reduce_agg_kernel(SumRows g, const float* pa, float* dAf, typename E::T* dAe, float c1) {
  using X = El<E>;
  int row, c;
  size_t first;
  const bool ok = g.place(row, c, first);
  f32x4 q = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < g.S; s0 += 8) {
    f32x4 x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = row4(pa, first + (size_t)min(s0 + k, g.S - 1) * g.n, g.d, c < g.d ? c : 0);
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (s0 + k < g.S) q += x[k];
  }
  if (!ok) return;
  const size_t o = (size_t)row * g.d + c;
  const f32x4 v = load_global<f32x4>(dAf + o) + q * c1;
  *reinterpret_cast<f32x4*>(dAf + o) = v;
  if (dAe) *reinterpret_cast<typename X::P4*>(dAe + o) = X::pack4(v[0], v[1], v[2], v[3]);
}

// ---------------------------------------------------------------------------
// dQ = round(dQ of the broadcast + Pooling^T(dA)) where the broadcast's kernel has left dQ in fp32: `src` ([units][N][d];
// null: dQ itself, in fp32).  dA = dAf + c1 * sum of the ranges of pa (S of them; none: dAf is complete) is finished here, in
// LDS, by every block of a unit.  A block takes 256 tokens: their places in the pooling grid are found once each (a dozen
// divisions), then a thread takes 16 bytes of a row.  Memory bounds it, most of all the way there: what a block reads is asked
// for ahead of everything else, all of it up to 32 channels (128 bytes of fp32 a thread; above, a turn for every 32).
// ---------------------------------------------------------------------------
struct PoolOutArgs {
  const float *src, *dAf, *pa;
  void* dQ;
  int S, N, n, d, gh, gw, ah, aw;
  uint32_t inv_cpr;      // of the 16-byte pieces in a row of dQ
  float c1;
  UnitPlace at;
};
template <class E>
__global__ __launch_bounds__(kThreads) void pool_grad_out_kernel(PoolOutArgs a) {
  using X = El<E>;
  using S = typename X::S;
  constexpr int kPer = X::kPerPiece, kBatch = 16 / kPer * 2;
  extern __shared__ __align__(16) unsigned char smem[];
  PoolPlace* place = reinterpret_cast<PoolPlace*>(smem);
  float* dA = reinterpret_cast<float*>(place + kThreads);
  const int u = blockIdx.y, tid = threadIdx.x, cpr = a.d / kPer, t0 = blockIdx.x * kThreads;
  const int pieces = min(kThreads, a.N - t0) * cpr;
  S* out = (S*)a.dQ + a.at.template base<kPer>(u, false);
  const float* src = a.src ? a.src + (size_t)u * a.N * a.d : nullptr;
  f32x4 v[kBatch][kPer / 4];
  S* at[kBatch];
  int tok[kBatch], c[kBatch];
  auto fetch = [&](int p0) {
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int p = min(p0 + k * kThreads, pieces - 1);
      tok[k] = quotient(p, a.inv_cpr);
      c[k] = (p - tok[k] * cpr) * kPer;
      at[k] = out + a.at.row(t0 + tok[k]) * a.at.sn + c[k];
#pragma unroll
      for (int h = 0; h < kPer / 4; ++h)
        v[k][h] = load_global<f32x4>((src ? src + (size_t)(t0 + tok[k]) * a.d + c[k] : (const float*)at[k]) + 4 * h);
    }
  };
  fetch(tid);
  const size_t nd = (size_t)a.n * a.d;
  for (int i = 4 * tid; i < (int)nd; i += 4 * kThreads) {
    const f32x4 own = load_global<f32x4>(a.dAf + (size_t)u * nd + i);
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < a.S; s0 += 8) {
      f32x4 x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = load_global<f32x4>(a.pa + ((size_t)u * a.S + min(s0 + k, a.S - 1)) * nd + i);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (s0 + k < a.S) sum += x[k];
    }
    *reinterpret_cast<f32x4*>(dA + i) = own + sum * a.c1;
  }
  const int mine = min(t0 + tid, a.N - 1), ty = mine / a.gw;
  place[tid].find(ty, mine - ty * a.gw, a.gh, a.gw, a.ah, a.aw);
  __syncthreads();
  for (int p0 = tid; p0 < pieces; p0 += kBatch * kThreads) {
    if (p0 != tid) fetch(p0);
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      if (p0 + k * kThreads >= pieces) continue;
      const PoolPlace pp = place[tok[k]];
#pragma unroll
      for (int h = 0; h < kPer / 4; ++h) v[k][h] += pp.gather(dA, a.d, c[k] + 4 * h);
      if constexpr (X::kBytes == 4) {
        *reinterpret_cast<f32x4*>(at[k]) = v[k][0];
      } else {
        const auto lo = X::pack4(v[k][0][0], v[k][0][1], v[k][0][2], v[k][0][3]);
        const auto hi = X::pack4(v[k][kPer / 4 - 1][0], v[k][kPer / 4 - 1][1], v[k][kPer / 4 - 1][2], v[k][kPer / 4 - 1][3]);
        *reinterpret_cast<u32x4*>(at[k]) = u32x4{lo[0], lo[1], hi[0], hi[1]};
      }
    }
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct FusedPlan {
  int DP, n_rows, ch_rows, token_cols, agent_cols[2], agent_blocks[2], S[2], chunk[2];      // [0]: agent kBc, [1]: kFwd / kAgg
  bool wide;
  bool both[2];      // one kernel takes the agents' and the tokens' gradients ([0]: kBc, [1]: kAgg)
  // agent bias, [0]: the broadcast's (B2), [1]: the aggregation's (B1); segments and pairs of columns as in AgentArgs
  bool bias[2];
  int cells[2], ld, segs[2], seg_len[2], pairs[2], per[2];
  // workspace offsets in floats (every region a multiple of 64 floats)
  size_t VAf, VAe, dVAe, lse1, w1, D1, lse2, w2, large, D2, dAf, dQf, part, total;
  bool weights[2];      // softmax rows may have a weight beside their reference
  size_t ta[2], tx[2], rows[2], yi[2], gt[2], gr[2], gsum[2], dwc;
};

size_t up64(size_t v) { return (v + 63) / 64 * 64; }

// forward: only what launch_forward_f32 needs
FusedPlan fused_plan(const Problem& p, bool forward = false) {
  FusedPlan f{};
  const bool f32 = p.dtype == 0;
  f.DP = p.d <= 32 ? 32 : (f32 && p.d <= 48 ? 48 : (p.d <= 64 ? 64 : (f32 && p.d <= 96 ? 96 : 128)));
  f.n_rows = (p.n + 31) / 32 * 32;      // the token kernels take agent tiles in pairs
  f.ch_rows = std::min(f.n_rows, f32 ? El<ElemF32>::kChunk : El<ElemBF16>::kChunk);
  f.bias[0] = p.b2.any(), f.bias[1] = p.b1.any();
  f.weights[0] = f32 || f.bias[0], f.weights[1] = f32 || f.bias[1];
  f.token_cols = f32 && f.DP > 64 ? 1 : 2;
  // token ranges: about two blocks per CU for the broadcast's agent kernel (192 registers) and with a bias, three for
  // the other two (which fit three blocks; four measured no faster).  At most kMaxRanges, which the merge's scale is made for.
  int groups[2];
  for (int k = 0; k < 2; ++k) {
    f.agent_cols[k] = (f32 || f.DP == 128 || p.n <= 64 || (k == 0 && f.bias[0] && f.DP == 64)) ? 1 : 2;
    const int per_block = 64 * f.agent_cols[k];      // agents per block
    f.agent_blocks[k] = (p.n + per_block - 1) / per_block;
    groups[k] = f.agent_blocks[k] * p.units;
    f.ld = std::max(f.ld, f.agent_blocks[k] * per_block);
    int S = ((2 + k) * kComputeUnits + groups[k] - 1) / groups[k];
    S = std::max(std::min(std::min(S, kMaxRanges), (p.N + 127) / 128), 1);
    f.chunk[k] = ((p.N + S - 1) / S + 31) / 32 * 32;
    f.S[k] = (p.N + f.chunk[k] - 1) / f.chunk[k];
  }
  f.cells[0] = p.b2.blk ? p.b2.h0 : 1, f.cells[1] = p.b1.blk ? p.b1.h0 : 1;
  const int xts = (p.gw + 15) / 16;
  for (int k = 0; k < 2; ++k) {
    if (!f.bias[k]) continue;
    // the ranges are pairs of columns: enough segments of at least four image rows for the number of ranges wanted,
    // an even number of columns, ranges of equally many pairs
    const int want = std::max(std::min((2 * kComputeUnits + groups[k] - 1) / groups[k], kMaxRanges), 1);
    int segs = std::max(1, std::min((2 * want + xts - 1) / xts, p.gh / 4));
    if (xts % 2 == 1 && segs % 2 == 1 && segs < p.gh) ++segs;
    f.seg_len[k] = (p.gh + segs - 1) / segs;
    f.segs[k] = (p.gh + f.seg_len[k] - 1) / f.seg_len[k];
    f.pairs[k] = (xts * f.segs[k] + 1) / 2;
    f.per[k] = (f.pairs[k] + want - 1) / want;
    f.S[k] = (f.pairs[k] + f.per[k] - 1) / f.per[k];
  }
  // four token columns per wave in the broadcast's token kernels when the unit has more than one 64-agent chunk to
  // reuse them on and that still leaves two blocks per CU
  f.wide = !f32 && f.DP <= 64 && p.n > 64 && (long long)((p.N + 255) / 256) * p.units >= 2 * kComputeUnits;
  // One kernel for both sides wherever a block of four waves holds all agents of a unit and the registers suffice (105
  // training steps of 8 .. 192 units of 196 .. 10000 tokens x 16 .. 64 agents, start / now: 0.73 to 0.97 of the time, 0.90 in the
  // mean).  Not dK / dV with a bias at 128 channels in 16 bits (263 registers spilled: 16 x 4 units of 784 x 16 285 -> 299 us) nor
  // fp32 above 64; the convolution without a bias is the token kernel's (its tokens are not walked down columns here), and so is
  // the residual with a bias and no convolution (a path for it beside the convolution's cost the latter 1 to 2 %).  From 2^30
  // elements on (16 bits) the broadcast's tokens stay with their own kernel, dQ in fp32 beside tensors of that size being 4 GiB
  // and more of workspace (time is not why: 256 units of 16384 x 49, d = 64, 2^28 elements, 2805 -> 2547 us).
  const bool room = f32 || (unsigned long long)p.units * p.N * p.d < 1ull << 30;
  for (int k = 0; k < 2; ++k)
    f.both[k] = !forward && p.n <= 64 && (!f32 || f.DP <= 64) && (k == 0 ? room : f.bias[1] ? (f32 || f.DP <= 64) && (p.dwc_w || p.vk == 0.0f) : !p.dwc_w);
  const size_t u = (size_t)p.units, nd = up64((size_t)p.n * p.d), un = up64(u * p.n), uN = up64(u * p.N);
  size_t o = 0;
  f.VAf = o, o += u * nd;
  f.VAe = f32 ? f.VAf : o, o += f32 ? 0 : u * nd / 2;
  f.lse1 = o, o += un;
  const size_t parts = (size_t)std::max(forward ? 0 : f.S[0], f.S[1]);
  f.part = o, o += up64(u * parts * p.n * (size_t)((forward ? 1 : 2) * p.d + 2));
  if (!forward) {
    f.dVAe = o, o += f32 ? u * nd : u * nd / 2;
    f.D1 = o, o += un;
    f.lse2 = o, o += uN;
    if (f.weights[1]) f.w1 = o, o += un;
    if (f.weights[0]) f.w2 = o, o += uN;
    if (!f32 && (f.bias[0] || f.bias[1])) f.large = o, o += up64(2 * u);
    f.D2 = o, o += uN;
    f.dAf = o, o += u * nd;
    if (f.both[0] && !f32 && p.ah > 0) f.dQf = o, o += up64(u * p.N * p.d);      // (no agent grid, no pooling term to wait for)
  }
  const size_t H = (size_t)p.heads, wp = 16 * (size_t)xts;
  for (int k = 0; k < 2; ++k) {
    if (!f.bias[k]) continue;
    const size_t table = up64(H * f.cells[k] * f.ld * wp);
    f.ta[k] = o, o += table;
    f.tx[k] = o, o += table;
    f.rows[k] = o, o += up64(H * p.gh * f.ld);
    f.yi[k] = o, o += up64((size_t)4 * p.gh);
    if (forward) continue;
    f.gt[k] = o, o += up64(u * f.segs[k] * f.cells[k] * f.ld * wp);
    f.gr[k] = o, o += up64(u * xts * p.gh * f.ld);
    f.gsum[k] = o, o += table;
  }
  if (p.dwc_w && !forward) f.dwc = o, o += up64(dwc_param_part_floats(p));
  f.total = o;
  return f;
}

// k: of the ranges, as in FusedPlan
SumRows sum_rows(const Problem& p, const FusedPlan& f, int k, dim3& grid) {
  SumRows g{p.units * p.n, p.n, p.d, f.S[k], 0};
  while ((4 << g.lpr_log2) < p.d) ++g.lpr_log2;
  const int per = kThreads >> g.lpr_log2;
  grid = dim3((g.rows + per - 1) / per);
  return g;
}

// Everything a pass launches: the tables of the biases in use and the token and agent kernels on top of them.
template <class E>
struct Pass {
  using T = typename E::T;
  const Problem& p;
  const FusedPlan& f;
  float* ws;
  hipStream_t st;
  float* w1;                  // where the agents' softmax rows leave their weights (null: they have none)
  int* large;                 // [2][units], of the tokens' and the agents' rows (null: no kernel asks)
  BiasTables bt[2] = {};

  hipError_t tables() {
    for (int k = 0; k < 2; ++k) {
      if (!f.bias[k]) continue;
      const bool has_rows = k == 0 ? p.b2.row != nullptr : p.b1.row != nullptr;
      float* rows = has_rows ? ws + f.rows[k] : nullptr;
      YInfo* yi = reinterpret_cast<YInfo*>(ws + f.yi[k]);
      bt[k] = BiasTables{ws + f.ta[k], ws + f.tx[k], rows, yi, f.cells[k], f.ld};
    }
    return launch_backward_bias_tables(p, bt, f.bias, large, large ? 2 * p.units : 0, st);
  }
  hipError_t token(int prob, TokenArgs& a) {
    const int k = prob == kAgg ? 1 : 0;
    a.ch_rows = f.bias[k] && prob == kBcStat ? std::min(f.ch_rows, chunk_rows<E, kBcStat, true>()) : f.ch_rows;
    const size_t lds = (size_t)2 * a.ch_rows * (f.DP + El<E>::kRowPad) * sizeof(T) + (size_t)3 * a.ch_rows * sizeof(float);
    if (f.bias[k]) {
      a.bt = bt[k];
      const int items = ((p.gw + 15) / 16) * ((p.gh + f.token_cols - 1) / f.token_cols);
      return launch_token<E, true>(prob, f.DP, f.token_cols, a, dim3((items + 3) / 4, p.units),
                                   lds + (size_t)4 * f.token_cols * a.ch_rows * sizeof(float), st);
    }
    const int cols = f.wide && prob != kAgg ? 4 : f.token_cols;
    return launch_token<E, false>(prob, f.DP, cols, a, dim3((p.N + 64 * cols - 1) / (64 * cols), p.units), lds, st);
  }
  // gt, gr: where the parts of the bias gradients go (null: not wanted)
  hipError_t agent(int prob, AgentArgs& a, float* gt, float* gr) {
    const int k = prob == kBc ? 0 : 1;
    const size_t lds = (size_t)4 * 32 * (f.DP + El<E>::kRowPad) * sizeof(T) + 2 * 96 * sizeof(float);
    const dim3 grid(f.S[k], f.agent_blocks[k], p.units);
    a.chunk = f.chunk[k], a.S = f.S[k];
    const bool both = prob != kFwd && f.both[k];
    if (!f.bias[k]) return both ? launch_both<E, false>(prob, f.DP, a, grid, lds, st) : launch_agent<E, false>(prob, f.DP, f.agent_cols[k], a, grid, lds, st);
    a.bt = bt[k], a.segs = f.segs[k], a.seg_len = f.seg_len[k], a.pairs = f.pairs[k], a.per = f.per[k];
    a.gt = gt, a.gr = gr;
    if (both) return launch_both<E, true>(prob, f.DP, a, grid, lds, st);
    return launch_agent<E, true>(prob, f.DP, f.agent_cols[k], a, grid, lds, st);
  }
  AgentArgs agent_args() const {
    AgentArgs a{};
    a.N = p.N, a.n = p.n, a.d = p.d, a.at = UnitPlace::make(p.lay, p.heads, El<E>::kBytes == 4 ? 2 : 3), a.gh = p.gh, a.gw = p.gw;
    return a;
  }
  TokenArgs token_args() const {
    TokenArgs a{};
    a.N = p.N, a.n = p.n, a.d = p.d, a.n_rows = f.n_rows, a.ch_rows = f.ch_rows, a.at = UnitPlace::make(p.lay, p.heads, El<E>::kBytes == 4 ? 2 : 3);
    a.gh = p.gh, a.gw = p.gw, a.ah = p.ah, a.aw = p.aw;
    return a;
  }
  // the aggregation: V_A (fp32 and element type) and the log-sum-exp of its rows
  hipError_t aggregate(const void* K, const void* V, const void* A) {
    float* part = ws + f.part;
    float* pm = part + (size_t)p.units * f.S[1] * p.n * p.d;
    float* pl = pm + (size_t)p.units * f.S[1] * p.n;
    AgentArgs a = agent_args();
    a.X = K, a.Y = V, a.M1 = A, a.P1 = part, a.pm = pm, a.pl = pl, a.sc = p.scale1 * kLog2e;
    const hipError_t e = agent(kFwd, a, nullptr, nullptr);
    if (e != hipSuccess) return e;
    dim3 grid;
    const SumRows g = sum_rows(p, f, 1, grid);
    fused_merge_kernel<E><<<grid, dim3(kThreads), 0, st>>>(g, part, pm, pl, ws + f.VAf, reinterpret_cast<T*>(ws + f.VAe),
                                                           ws + f.lse1, w1, large && f.bias[1] ? large + p.units : nullptr);
    return hipGetLastError();
  }
};

template <class E>
hipError_t run_fused(const Problem& p, const FusedPlan& f, const void* Q, const void* K, const void* V, const void* A,
                     const void* dO, float* ws, void* dQ, void* dK, void* dV, void* dA, bool agents_given,
                     const BackwardParamGrads& pg, hipStream_t st) {
  using T = typename E::T;
  const int U = p.units, n = p.n, d = p.d;
  float* VAf = ws + f.VAf;
  T* VAe = reinterpret_cast<T*>(ws + f.VAe);
  T* dVAe = reinterpret_cast<T*>(ws + f.dVAe);
  float *lse1 = ws + f.lse1, *D1 = ws + f.D1, *lse2 = ws + f.lse2, *D2 = ws + f.D2, *dAf = ws + f.dAf;
  float* part1 = ws + f.part;
  float* part2 = part1 + (size_t)U * f.S[0] * n * d;      // kBc only
  const float sc1 = p.scale1 * kLog2e, sc2 = p.scale2 * kLog2e;
  float *w1 = f.weights[1] ? ws + f.w1 : nullptr, *w2 = f.weights[0] ? ws + f.w2 : nullptr;
  int* large = El<E>::kBytes == 2 && (f.bias[0] || f.bias[1]) ? reinterpret_cast<int*>(ws + f.large) : nullptr;
  Pass<E> pass{p, f, ws, st, w1, large};
  hipError_t e = pass.tables();
  if (e != hipSuccess) return e;
  // the aggregation again
  if ((e = pass.aggregate(K, V, A)) != hipSuccess) return e;

  // broadcast: per-token row statistics, then the per-agent sums
  AgentArgs ag = pass.agent_args();
  TokenArgs tk = pass.token_args();
  tk.X = Q, tk.Y = dO, tk.M1 = A, tk.M2 = VAe, tk.st1 = lse2, tk.st2 = D2, tk.sc = sc2, tk.oscale = p.scale2;
  tk.st3 = w2, ag.tw1 = w2, tk.rw1 = ag.rw1 = w1, tk.large = large, ag.large = large;
  if ((e = pass.token(kBcStat, tk)) != hipSuccess) return e;
  ag.X = Q, ag.Y = dO, ag.M1 = A, ag.M2 = VAe, ag.ts1 = lse2, ag.ts2 = D2, ag.P1 = part1, ag.P2 = part2, ag.sc = sc2;
  float* dQf = f.both[0] && !agents_given && El<E>::kBytes == 2 ? ws + f.dQf : nullptr;
  ag.O1 = dQ, ag.Of = dQf, ag.oscale = p.scale2;
  if ((e = pass.agent(kBc, ag, pg.db2_col || pg.db2_blk ? ws + f.gt[0] : nullptr, pg.db2_row ? ws + f.gr[0] : nullptr)) !=
      hipSuccess)
    return e;
  dim3 rgrid;
  const SumRows rows_bc = sum_rows(p, f, 0, rgrid);
  fused_reduce_bc_kernel<E><<<rgrid, dim3(kThreads), 0, st>>>(rows_bc, part1, part2, VAf, dVAe, D1, dAf, p.scale2);

  // aggregation
  if (large) tk.large = large + U, ag.large = large + U;
  tk.X = K, tk.Y = V, tk.M2 = dVAe, tk.rs1 = lse1, tk.rs2 = D1, tk.sc = sc1, tk.oscale = p.scale1;
  tk.O1 = dK, tk.O2 = dV, tk.G = dO, tk.vk = p.vk, tk.dwc_w = p.dwc_w;
  if (!f.both[1] && (e = pass.token(kAgg, tk)) != hipSuccess) return e;
  ag.O1 = dK, ag.O2 = dV, ag.Of = nullptr, ag.oscale = p.scale1, ag.G = dO, ag.vk = p.vk, ag.dwc_w = p.dwc_w;
  ag.X = K, ag.Y = V, ag.M2 = dVAe, ag.rs1 = lse1, ag.rs2 = D1, ag.P1 = part1, ag.sc = sc1;
  if ((e = pass.agent(kAgg, ag, pg.db1_col || pg.db1_blk ? ws + f.gt[1] : nullptr, pg.db1_row ? ws + f.gr[1] : nullptr)) !=
      hipSuccess)
    return e;
  // dQ last: the pooling term needs the finished dA
  if (f.both[0] && !agents_given) {
    // many ranges (few units): added up first, not by every block
    const bool sum_first = f.S[1] > 8;
    if (sum_first) {
      const SumRows rows_agg = sum_rows(p, f, 1, rgrid);
      fused_reduce_agg_kernel<E><<<rgrid, dim3(kThreads), 0, st>>>(rows_agg, part1, dAf, (T*)nullptr, p.scale1);
    }
    PoolOutArgs po{};
    po.src = dQf, po.dAf = dAf, po.pa = part1, po.dQ = dQ, po.S = sum_first ? 0 : f.S[1], po.N = p.N, po.n = n, po.d = d;
    po.gh = p.gh, po.gw = p.gw, po.ah = p.ah, po.aw = p.aw, po.c1 = p.scale1, po.at = tk.at;
    po.inv_cpr = quotient_inverse(d / El<E>::kPerPiece);
    const size_t lds = kThreads * sizeof(PoolPlace) + (size_t)n * d * sizeof(float);
    pool_grad_out_kernel<E><<<dim3((p.N + kThreads - 1) / kThreads, U), dim3(kThreads), lds, st>>>(po);
    e = hipGetLastError();
  } else {
    const SumRows rows_agg = sum_rows(p, f, 1, rgrid);
    fused_reduce_agg_kernel<E><<<rgrid, dim3(kThreads), 0, st>>>(rows_agg, part1, dAf, agents_given ? (T*)dA : nullptr, p.scale1);
    tk.large = large;
    tk.X = Q, tk.Y = dO, tk.M2 = VAe, tk.sc = sc2, tk.oscale = p.scale2, tk.O1 = dQ, tk.dA = agents_given ? nullptr : dAf;
    if (!f.both[0]) e = pass.token(kBc, tk);
  }
  if (e != hipSuccess) return e;

  BiasGradParts parts[2] = {};
  for (int k = 0; k < 2; ++k)
    if (f.bias[k]) parts[k] = BiasGradParts{ws + f.gt[k], ws + f.gr[k], ws + f.gsum[k], f.segs[k], f.seg_len[k], f.cells[k], f.ld};
  return launch_backward_param_grads(p, parts, pg, V, dO, ws + f.dwc, st);
}

}  // namespace

// places within a unit in 32 bits (see UnitPlace::fits); fp32 units past them have another path
static bool short_units(const Problem& p) { return p.dtype == 0 || p.b1.any() || p.b2.any() || p.dwc_w; }

bool backward_fused_supported(const Problem& p) {
  return p.d % (p.dtype == 0 ? 4 : 8) == 0 && p.d <= 128 && p.units <= 65535 &&
         (unsigned long long)p.N * p.d * p.heads >> 34 == 0 && (!short_units(p) || (unsigned long long)p.N * p.d < (1ull << 30));
}

bool fused_layout_supported(const Problem& p) {
  const int m = p.dtype == 0 ? 4 : 8;      // 16-byte rows
  const Layout& l = p.lay;
  return l.sb % m == 0 && l.sh % m == 0 && l.sn % m == 0 && l.ob % m == 0 && l.oh % m == 0 && l.on % m == 0 &&
         UnitPlace::fits(l, p.N, short_units(p));
}

size_t backward_fused_workspace_floats(const Problem& p) { return fused_plan(p).total; }

hipError_t launch_backward_fused(const Problem& p, const void* Q, const void* K, const void* V, const void* A_elem,
                                 const void* dO, float* ws, void* dQ, void* dK, void* dV, void* dA, bool agents_given,
                                 const BackwardParamGrads& pg, hipStream_t st) {
  const FusedPlan f = fused_plan(p);
  if (p.dtype == 2) return run_fused<ElemBF16>(p, f, Q, K, V, A_elem, dO, ws, dQ, dK, dV, dA, agents_given, pg, st);
  if (p.dtype == 1) return run_fused<ElemF16>(p, f, Q, K, V, A_elem, dO, ws, dQ, dK, dV, dA, agents_given, pg, st);
  return run_fused<ElemF32>(p, f, Q, K, V, A_elem, dO, ws, dQ, dK, dV, dA, agents_given, pg, st);
}

// ---------------------------------------------------------------------------
// Forward pass of fp32 problems that the one-launch kernel does not serve (more agents or tokens than fit in LDS, an
// agent bias): the aggregation as in the backward pass, then the token kernel's broadcast.
// ---------------------------------------------------------------------------
bool forward_f32_supported(const Problem& p) { return p.dtype == 0 && backward_fused_supported(p); }

size_t forward_f32_workspace_floats(const Problem& p) { return fused_plan(p, true).total; }

hipError_t launch_forward_f32(const Problem& p, const void* Q, const void* K, const void* V, const void* A, float* ws,
                              void* out, hipStream_t st) {
  const FusedPlan f = fused_plan(p, true);
  Pass<ElemF32> pass{p, f, ws, st, nullptr, nullptr};
  hipError_t e = pass.tables();
  if (e != hipSuccess) return e;
  if ((e = pass.aggregate(K, V, A)) != hipSuccess) return e;
  TokenArgs tk = pass.token_args();
  tk.X = tk.Y = Q, tk.M1 = A, tk.M2 = ws + f.VAe, tk.sc = p.scale2 * kLog2e, tk.O1 = out;
  tk.G = V, tk.vk = p.vk, tk.dwc_w = p.dwc_w, tk.dwc_b = p.dwc_b;
  return pass.token(kOut, tk);
}

}  // namespace aa
