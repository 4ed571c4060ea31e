// Recomputing backward (backward_fused.inc): the kernels without an agent bias, the sums over the token ranges and the
// host side.
#include "backward_fused.inc"

#include <algorithm>

namespace aa {

// compiled by backward_bias_{bf16,f16}.hip
extern template hipError_t launch_token_bias<ElemBF16>(int, int, const TokenArgs&, dim3, size_t, hipStream_t);
extern template hipError_t launch_token_bias<ElemF16>(int, int, const TokenArgs&, dim3, size_t, hipStream_t);
extern template hipError_t launch_agent_bias<ElemBF16>(int, int, int, const AgentArgs&, dim3, size_t, hipStream_t);
extern template hipError_t launch_agent_bias<ElemF16>(int, int, int, const AgentArgs&, dim3, size_t, hipStream_t);

namespace {

// ---------------------------------------------------------------------------
// Sums over the token ranges, one 64-lane block per (agent, unit), lane = channel (and channel + 64), ranges
// in order.
// ---------------------------------------------------------------------------
// log-sum-exp merge of the recomputed aggregation: V_A (fp32 and element type) and lse1 (log2 domain)
template <class E>
__global__ __launch_bounds__(64) void fused_merge_kernel(const float* __restrict__ acc, const float* __restrict__ pm,
                                                         const float* __restrict__ pl, int S, int n, int d,
                                                         float* __restrict__ VAf, uint16_t* __restrict__ VAe,
                                                         float* __restrict__ lse1) {
  const int ag = blockIdx.x, u = blockIdx.y, lane = threadIdx.x;
  __shared__ float wgt[64];
  // lane s holds range s (S <= 64)
  const size_t my = ((size_t)u * S + min(lane, S - 1)) * n + ag;
  const float pm_s = lane < S ? pm[my] : -INFINITY, pl_s = lane < S ? pl[my] : 0.f;
  const float M = wave_max(pm_s);
  const float w_s = fast_exp2(pm_s - M);
  const float L = wave_sum(pl_s * w_s);
  wgt[lane] = w_s / L;
  __syncthreads();
  for (int c = lane; c < d; c += 64) {
    float v = 0.f;
    for (int s = 0; s < S; ++s) v += acc[(((size_t)u * S + s) * n + ag) * d + c] * wgt[s];
    const size_t o = ((size_t)u * n + ag) * d + c;
    VAf[o] = v;
    const typename E::T e = E::from_f32(v);
    VAe[o] = __builtin_bit_cast(uint16_t, e);
  }
  if (lane == 0) lse1[(size_t)u * n + ag] = M + __builtin_amdgcn_logf(L);
}

// dV_A = sum of the ranges (element type), D1 = rowsum(dV_A o V_A), dA = c2 * sum of the ranges
template <class E>
__global__ __launch_bounds__(64) void fused_reduce_bc_kernel(const float* __restrict__ pva, const float* __restrict__ pa,
                                                             int S, int n, int d, const float* __restrict__ VAf,
                                                             uint16_t* __restrict__ dVAe, float* __restrict__ D1,
                                                             float* __restrict__ dAf, float c2) {
  const int ag = blockIdx.x, u = blockIdx.y, lane = threadIdx.x;
  float dot = 0.f;
  for (int c = lane; c < d; c += 64) {
    float v = 0.f, q = 0.f;
    for (int s = 0; s < S; ++s) {
      const size_t i = (((size_t)u * S + s) * n + ag) * d + c;
      v += pva[i];
      q += pa[i];
    }
    const size_t o = ((size_t)u * n + ag) * d + c;
    const typename E::T e = E::from_f32(v);
    dVAe[o] = __builtin_bit_cast(uint16_t, e);
    dot += E::to_f32(e) * VAf[o];
    dAf[o] = c2 * q;
  }
  dot = wave_sum(dot);
  if (lane == 0) D1[(size_t)u * n + ag] = dot;
}

// dA += c1 * sum of the ranges; written in the element type too when the agents were handed in
template <class E>
__global__ __launch_bounds__(64) void fused_reduce_agg_kernel(const float* __restrict__ pa, int S, int n, int d,
                                                              float* __restrict__ dAf, uint16_t* __restrict__ dAe, float c1) {
  const int ag = blockIdx.x, u = blockIdx.y, lane = threadIdx.x;
  for (int c = lane; c < d; c += 64) {
    float q = 0.f;
    for (int s = 0; s < S; ++s) q += pa[(((size_t)u * S + s) * n + ag) * d + c];
    const size_t o = ((size_t)u * n + ag) * d + c;
    const float v = dAf[o] + c1 * q;
    dAf[o] = v;
    if (dAe) {
      const typename E::T e = E::from_f32(v);
      dAe[o] = __builtin_bit_cast(uint16_t, e);
    }
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct FusedPlan {
  int DP, n_rows, ch_rows, agent_cols, agent_blocks, S[2], chunk[2];      // [0]: agent kBc, [1]: agent kFwd / kAgg
  bool wide;
  // agent bias, [0]: the broadcast's (B2), [1]: the aggregation's (B1); segments and pairs of columns as in AgentArgs
  bool bias[2];
  int cells[2], ld, segs[2], seg_len[2], pairs[2], per[2];
  // workspace offsets in floats (every region a multiple of 64 floats)
  size_t VAf, VAe, dVAe, lse1, D1, lse2, D2, dAf, part, total;
  size_t ta[2], tx[2], rows[2], gt[2], gr[2], gsum[2], dwc;
};

size_t up64(size_t v) { return (v + 63) / 64 * 64; }

FusedPlan fused_plan(const Problem& p) {
  FusedPlan f{};
  f.DP = p.d <= 32 ? 32 : (p.d <= 64 ? 64 : 128);
  f.n_rows = (p.n + 31) / 32 * 32;      // the token kernels take agent tiles in pairs
  f.ch_rows = min(f.n_rows, 128);
  f.agent_cols = (f.DP == 128 || p.n <= 64) ? 1 : 2;
  const int per_block = 64 * f.agent_cols;      // agents per block of the agent kernels
  f.agent_blocks = (p.n + per_block - 1) / per_block;
  const int groups = f.agent_blocks * p.units;
  // token ranges: about two blocks per CU for the broadcast's agent kernel (192 registers), three for the other
  // two (which fit three blocks; four measured no faster).  At most 64: the merge gives every range a lane.
  for (int k = 0; k < 2; ++k) {
    int S = ((2 + k) * kComputeUnits + groups - 1) / groups;
    S = max(min(min(S, 64), (p.N + 127) / 128), 1);
    f.chunk[k] = ((p.N + S - 1) / S + 31) / 32 * 32;
    f.S[k] = (p.N + f.chunk[k] - 1) / f.chunk[k];
  }
  f.bias[0] = p.b2.any(), f.bias[1] = p.b1.any();
  f.cells[0] = p.b2.blk ? p.b2.h0 : 1, f.cells[1] = p.b1.blk ? p.b1.h0 : 1;
  f.ld = std::max((p.n + 63) / 64 * 64, f.agent_blocks * per_block);
  const int xts = (p.gw + 15) / 16;
  for (int k = 0; k < 2; ++k) {
    if (!f.bias[k]) continue;
    // the ranges are pairs of columns: enough segments of at least four image rows for the number of ranges wanted,
    // an even number of columns, ranges of equally many pairs
    const int want = std::max(std::min((2 * kComputeUnits + groups - 1) / groups, 64), 1);
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
  f.wide = f.DP <= 64 && p.n > 64 && (long long)((p.N + 255) / 256) * p.units >= 2 * kComputeUnits;
  const size_t u = (size_t)p.units, nd = up64((size_t)p.n * p.d), un = up64(u * p.n), uN = up64(u * p.N);
  size_t o = 0;
  f.VAf = o, o += u * nd;
  f.VAe = o, o += u * nd / 2;
  f.dVAe = o, o += u * nd / 2;
  f.lse1 = o, o += un;
  f.D1 = o, o += un;
  f.lse2 = o, o += uN;
  f.D2 = o, o += uN;
  f.dAf = o, o += u * nd;
  f.part = o, o += up64(u * max(f.S[0], f.S[1]) * p.n * (size_t)(2 * p.d + 2));
  const size_t H = (size_t)p.heads, wp = 16 * (size_t)xts;
  for (int k = 0; k < 2; ++k) {
    if (!f.bias[k]) continue;
    const size_t table = up64(H * f.cells[k] * f.ld * wp);
    f.ta[k] = o, o += table;
    f.tx[k] = o, o += table;
    f.rows[k] = o, o += up64(H * p.gh * f.ld);
    f.gt[k] = o, o += up64(u * f.segs[k] * f.cells[k] * f.ld * wp);
    f.gr[k] = o, o += up64(u * xts * p.gh * f.ld);
    f.gsum[k] = o, o += table;
  }
  if (p.dwc_w) f.dwc = o, o += up64(dwc_param_part_floats(p));
  f.total = o;
  return f;
}

template <class E, int DP>
hipError_t run_fused(const Problem& p, const FusedPlan& f, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                     const uint16_t* A, const uint16_t* dO, float* ws, void* dQ, void* dK, void* dV, void* dA,
                     bool agents_given, const BackwardParamGrads& pg, hipStream_t st) {
  using G = Geo<DP>;
  const int U = p.units, N = p.N, n = p.n, d = p.d;
  float* VAf = ws + f.VAf;
  uint16_t* VAe = reinterpret_cast<uint16_t*>(ws + f.VAe);
  uint16_t* dVAe = reinterpret_cast<uint16_t*>(ws + f.dVAe);
  float *lse1 = ws + f.lse1, *D1 = ws + f.D1, *lse2 = ws + f.lse2, *D2 = ws + f.D2, *dAf = ws + f.dAf;
  float* part1 = ws + f.part;
  float* part2 = part1 + (size_t)U * f.S[0] * n * d;      // kBc only
  float* pm = part1 + (size_t)U * f.S[1] * n * d;         // kFwd only
  float* pl = pm + (size_t)U * f.S[1] * n;
  const float sc1 = p.scale1 * kLog2e, sc2 = p.scale2 * kLog2e;

  const size_t agent_lds = (size_t)4 * 32 * G::LST * 2 + 2 * 64 * sizeof(float);
  const size_t token_lds = (size_t)2 * f.ch_rows * G::LST * 2 + (size_t)2 * f.ch_rows * sizeof(float);
  const size_t token_bias_lds = token_lds + (size_t)4 * kBiasTokenCols * f.ch_rows * sizeof(float);
  const dim3 rgrid(n, U);
  constexpr int NW = DP <= 64 ? 4 : 2;      // the wide form is never chosen at DP = 128
  constexpr int C2 = DP <= 64 ? 2 : 1;
  hipError_t e = hipSuccess;

  // bias tables of the kinds in use
  BiasTables bt[2] = {};
  for (int k = 0; k < 2; ++k) {
    if (!f.bias[k]) continue;
    const bool has_rows = k == 0 ? p.b2.row != nullptr : p.b1.row != nullptr;
    bt[k] = BiasTables{ws + f.ta[k], ws + f.tx[k], has_rows ? ws + f.rows[k] : nullptr, f.cells[k], f.ld};
    e = launch_backward_bias_tables(p, k == 0 ? 2 : 1, f.cells[k], f.ld, ws + f.ta[k], ws + f.tx[k],
                                    has_rows ? ws + f.rows[k] : nullptr, st);
    if (e != hipSuccess) return e;
  }
  // one launch of a token / agent kernel, with or without its stage's bias
  auto token = [&](auto prob_c, TokenArgs& a) -> hipError_t {
    constexpr int PROB = decltype(prob_c)::value, k = PROB == kAgg ? 1 : 0;
    if (f.bias[k]) {
      a.bt = bt[k];
      const int items = ((p.gw + 15) / 16) * ((p.gh + kBiasTokenCols - 1) / kBiasTokenCols);
      return launch_token_bias<E>(PROB, DP, a, dim3((items + 3) / 4, U), token_bias_lds, st);
    }
    auto go = [&](auto kernel, int tokens) -> hipError_t {
      const hipError_t err = allow_lds(kernel, token_lds);
      if (err != hipSuccess) return err;
      kernel<<<dim3((N + tokens - 1) / tokens, U), dim3(kThreads), token_lds, st>>>(a);
      return hipGetLastError();
    };
    if constexpr (PROB != kAgg)
      if (f.wide) return go(fused_token_kernel<E, DP, PROB, NW, false>, 256);
    return go(fused_token_kernel<E, DP, PROB, 2, false>, 128);
  };
  auto agent = [&](auto prob_c, AgentArgs& a) -> hipError_t {
    constexpr int PROB = decltype(prob_c)::value, k = PROB == kBc ? 0 : 1;
    a.chunk = f.chunk[k], a.S = f.S[k];
    const dim3 grid(f.S[k], f.agent_blocks, U);
    if (f.bias[k]) {
      a.bt = bt[k], a.segs = f.segs[k], a.seg_len = f.seg_len[k], a.pairs = f.pairs[k], a.per = f.per[k];
      const bool cells = k == 0 ? pg.db2_col || pg.db2_blk : pg.db1_col || pg.db1_blk;
      a.gt = cells ? ws + f.gt[k] : nullptr;
      a.gr = (k == 0 ? pg.db2_row : pg.db1_row) ? ws + f.gr[k] : nullptr;
      return launch_agent_bias<E>(PROB, DP, f.agent_cols, a, grid, agent_lds, st);
    }
    if (f.agent_cols == 2)
      fused_agent_kernel<E, DP, PROB, C2, false><<<grid, dim3(kThreads), agent_lds, st>>>(a);
    else
      fused_agent_kernel<E, DP, PROB, 1, false><<<grid, dim3(kThreads), agent_lds, st>>>(a);
    return hipGetLastError();
  };
  using FwdC = std::integral_constant<int, kFwd>;
  using BcC = std::integral_constant<int, kBc>;
  using AggC = std::integral_constant<int, kAgg>;
  using StatC = std::integral_constant<int, kBcStat>;

  AgentArgs ag{};
  ag.N = N, ag.n = n, ag.d = d, ag.at = UnitPlace::make(p.lay, p.heads), ag.gh = p.gh, ag.gw = p.gw;
  // the aggregation again: V_A and the log-sum-exp of its rows
  ag.X = K, ag.Y = V, ag.M1 = A, ag.M2 = nullptr, ag.P1 = part1, ag.pm = pm, ag.pl = pl, ag.sc = sc1;
  if ((e = agent(FwdC{}, ag)) != hipSuccess) return e;
  fused_merge_kernel<E><<<rgrid, dim3(64), 0, st>>>(part1, pm, pl, f.S[1], n, d, VAf, VAe, lse1);

  // broadcast: per-token row statistics, then the per-agent sums
  TokenArgs tk{};
  tk.N = N, tk.n = n, tk.d = d, tk.n_rows = f.n_rows, tk.ch_rows = f.ch_rows, tk.at = ag.at;
  tk.gh = p.gh, tk.gw = p.gw, tk.ah = p.ah, tk.aw = p.aw;
  tk.X = Q, tk.Y = dO, tk.M1 = A, tk.M2 = VAe, tk.st1 = lse2, tk.st2 = D2, tk.sc = sc2, tk.oscale = p.scale2;
  if ((e = token(StatC{}, tk)) != hipSuccess) return e;
  ag.X = Q, ag.Y = dO, ag.M2 = VAe, ag.ts1 = lse2, ag.ts2 = D2, ag.P1 = part1, ag.P2 = part2, ag.sc = sc2;
  if ((e = agent(BcC{}, ag)) != hipSuccess) return e;
  fused_reduce_bc_kernel<E><<<rgrid, dim3(64), 0, st>>>(part1, part2, f.S[0], n, d, VAf, dVAe, D1, dAf, p.scale2);

  // aggregation
  tk.X = K, tk.Y = V, tk.M2 = dVAe, tk.rs1 = lse1, tk.rs2 = D1, tk.sc = sc1, tk.oscale = p.scale1;
  tk.O1 = dK, tk.O2 = dV, tk.G = dO, tk.vk = p.vk, tk.dwc_w = p.dwc_w;
  if ((e = token(AggC{}, tk)) != hipSuccess) return e;
  ag.X = K, ag.Y = V, ag.M2 = dVAe, ag.rs1 = lse1, ag.rs2 = D1, ag.P1 = part1, ag.sc = sc1;
  if ((e = agent(AggC{}, ag)) != hipSuccess) return e;
  fused_reduce_agg_kernel<E><<<rgrid, dim3(64), 0, st>>>(part1, f.S[1], n, d, dAf, agents_given ? (uint16_t*)dA : nullptr,
                                                         p.scale1);
  // dQ last: the pooling term needs the finished dA
  tk.X = Q, tk.Y = dO, tk.M2 = VAe, tk.sc = sc2, tk.oscale = p.scale2, tk.O1 = dQ, tk.dA = agents_given ? nullptr : dAf;
  if ((e = token(BcC{}, tk)) != hipSuccess) return e;

  // parameter gradients
  for (int k = 0; k < 2; ++k) {
    if (!f.bias[k]) continue;
    const BiasGradParts parts{ws + f.gt[k], ws + f.gr[k], ws + f.gsum[k], f.segs[k], f.seg_len[k], f.cells[k], f.ld};
    e = k == 0 ? launch_backward_bias_grads(p, 2, parts, pg.h0, pg.w0, pg.db2_col, pg.db2_row, pg.db2_blk, st)
               : launch_backward_bias_grads(p, 1, parts, pg.h0, pg.w0, pg.db1_col, pg.db1_row, pg.db1_blk, st);
    if (e != hipSuccess) return e;
  }
  if (p.dwc_w && pg.ddwc_w) return launch_dwc_param_grads(p, V, dO, ws + f.dwc, pg.ddwc_w, pg.ddwc_b, st);
  return hipGetLastError();
}

template <class E>
hipError_t run_fused_dp(const Problem& p, const FusedPlan& f, const void* Q, const void* K, const void* V, const void* A,
                        const void* dO, float* ws, void* dQ, void* dK, void* dV, void* dA, bool agents_given,
                        const BackwardParamGrads& pg, hipStream_t st) {
  const uint16_t *q = (const uint16_t*)Q, *k = (const uint16_t*)K, *v = (const uint16_t*)V, *a = (const uint16_t*)A,
                 *g = (const uint16_t*)dO;
  switch (f.DP) {
    case 32: return run_fused<E, 32>(p, f, q, k, v, a, g, ws, dQ, dK, dV, dA, agents_given, pg, st);
    case 64: return run_fused<E, 64>(p, f, q, k, v, a, g, ws, dQ, dK, dV, dA, agents_given, pg, st);
    default: return run_fused<E, 128>(p, f, q, k, v, a, g, ws, dQ, dK, dV, dA, agents_given, pg, st);
  }
}

}  // namespace

bool backward_fused_supported(const Problem& p) {
  return (p.dtype == 1 || p.dtype == 2) && p.d % 8 == 0 && p.d <= 128 && p.units <= 65535;
}

size_t backward_fused_workspace_floats(const Problem& p) { return fused_plan(p).total; }

hipError_t launch_backward_fused(const Problem& p, const void* Q, const void* K, const void* V, const void* A_elem,
                                 const void* dO, float* ws, void* dQ, void* dK, void* dV, void* dA, bool agents_given,
                                 const BackwardParamGrads& pg, hipStream_t st) {
  const FusedPlan f = fused_plan(p);
  if (p.dtype == 2) return run_fused_dp<ElemBF16>(p, f, Q, K, V, A_elem, dO, ws, dQ, dK, dV, dA, agents_given, pg, st);
  return run_fused_dp<ElemF16>(p, f, Q, K, V, A_elem, dO, ws, dQ, dK, dV, dA, agents_given, pg, st);
}

}  // namespace aa
