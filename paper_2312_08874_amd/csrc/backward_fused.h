// What the units of the recomputing backward share: kernel arguments, the agent-bias tables and the launchers.
#pragma once
#include "kernels.h"

namespace aa {

constexpr int kThreads = 256;       // four waves per block
enum { kFwd = 0, kBc = 1, kAgg = 2, kBcStat = 3, kOut = 4 };

// Agent bias of one kind as the recomputing kernels read it (fp32, times log2 e; see backward_fused.inc):
//   bias(a, (y, x)) = (1 - f) T[i][x][a] + f T[i + 1][x][a] + R[y][a]
// T in two orders, wp = gw rounded up to 16 (columns past gw hold a score mask), ld agents (n rounded up, zeros):
//   ta [heads][cells][ld / 4][wp][4 agents]     for lanes that hold a token and four agents
//   tx [heads][cells][wp / 4][ld][4 columns]    for lanes that hold an agent and four neighbours in x
// rows [heads][gh][ld], null when there is no row component.
// Entries of T and R are finite: below kBiasFloor (a mask of the type's lowest value or of minus infinity) they are that,
// so that differences of two masked entries are zero.  What does not exist (columns past gw, agents past n in the kernels)
// is kMaskedScore, far below the sum of two of them and still finite.
// yi [gh]: what an image row needs to know of the interpolation along y.
constexpr float kBiasFloor = -1.0e30f, kMaskedScore = -1.0e38f;
struct YInfo {
  int cell, next;      // cell row i; the first image row below with another one (or gh)
  float f;             // weight of cell row i + 1 (0 on the last cell row)
  int pad;
};
struct BiasTables {
  const float *ta, *tx, *rows;
  const YInfo* yi;
  int cells, ld;
};

// Where a unit's rows start and which row a token is: Layout for the recomputing kernels, with 32-bit strides (in 16-byte
// pieces of 1 << piece_log2 elements), every division a multiplication and the windows behind one branch (at 10 us a kernel
// the scalar instructions ahead of its first load show).
struct UnitPlace {
  uint32_t sb, sh, ob, oh;
  int sn, on, heads, line;
  uint32_t inv_heads, inv_nwin, inv_wxn, inv_ww;         // ceil(2^32 / divisor), 0 for a divisor of 1 (inv_ww: no windows)
  int nwin, wxn, ww, win_rows;                           // win_rows: image rows of a window times line

  static unsigned long long rows(const Layout& l, int N) { return l.line ? (unsigned long long)l.wh * l.line : (unsigned long long)N; }
  // strides below 2^34 elements, windows only where N * ww < 2^32; short_units: a unit's extent below 2^32 bytes, for the
  // kernels with a bias and the convolution, which keep their places within a unit in 32 bits
  static bool fits(const Layout& l, int N, bool short_units) {
    return ((unsigned long long)l.sb | (unsigned long long)l.sh | (unsigned long long)l.ob | (unsigned long long)l.oh) >> 34 == 0 &&
           (l.line == 0 || (unsigned long long)N * l.ww >> 32 == 0) &&
           (!short_units || (rows(l, N) * (unsigned long long)l.sn >> 30 == 0 && rows(l, N) * (unsigned long long)l.on >> 30 == 0));
  }
  static UnitPlace make(const Layout& l, int heads, int piece_log2) {
    UnitPlace p{};
    p.sb = (uint32_t)(l.sb >> piece_log2), p.sh = (uint32_t)(l.sh >> piece_log2);
    p.ob = (uint32_t)(l.ob >> piece_log2), p.oh = (uint32_t)(l.oh >> piece_log2);
    p.sn = l.sn, p.on = l.on, p.heads = heads, p.line = l.line;
    p.nwin = l.nwin, p.wxn = l.wxn, p.ww = l.line ? l.ww : 0, p.win_rows = l.wh * l.line;
    p.inv_heads = quotient_inverse(heads), p.inv_nwin = quotient_inverse(l.nwin), p.inv_wxn = quotient_inverse(l.wxn);
    p.inv_ww = l.line ? quotient_inverse(l.ww) : 0u;
    return p;
  }
  __device__ __forceinline__ int entry(int u) const { return quotient(u, inv_heads); }
  template <int kPiece>
  __device__ __forceinline__ size_t base(int u, bool out) const {
    const uint32_t bw = entry(u), hd = u - bw * heads;
    uint32_t b = bw;
    size_t at = 0;
    if (line != 0) {
      b = quotient(bw, inv_nwin);
      const int win = bw - b * nwin, wy = quotient(win, inv_wxn), wx = win - wy * wxn;
      at += ((size_t)wy * (size_t)win_rows + (size_t)(wx * ww)) * (size_t)(out ? on : sn);
    }
    return at + ((size_t)hd * (out ? oh : sh) + (size_t)b * (out ? ob : sb)) * kPiece;
  }
  __device__ __forceinline__ size_t row(int t) const {
    if (line == 0) return (size_t)t;
    const int y = quotient(t, inv_ww);
    return (size_t)t + (size_t)((long long)y * (line - ww));
  }
  __device__ __forceinline__ int pitch(int gw) const { return line == 0 ? gw : line; }
};

struct TokenArgs {
  const void *X, *Y, *M1, *M2;      // in the element type
  const float *rs1, *rs2, *rw1;      // reference, D1 and weight of the agents' softmax rows
  float *st1, *st2, *st3;            // of the tokens': reference, D2, weight
  int* large;                        // 16 bits with a bias: per unit, whether one of these rows has a large reference
  void *O1, *O2;
  int N, n, d, n_rows, ch_rows;      // n_rows: n rounded up to 32; ch_rows: agents staged at a time (x32)
  const float* dA;                   // kBc: the finished dA [units][n][d] when the agents were pooled (else null)
  int gh, gw, ah, aw;                // token grid, the pooling's agent grid
  float sc, oscale;
  const void* G;          // kAgg: dO, for the share of dV that comes through the V residual (Appendix C.1: O += k V)
  float vk;               //   and through the depthwise convolution (Eq. (6), dwc_w [heads][d][3][3] or null);
  const float* dwc_w;     //   kOut: V, for these terms themselves
  const float* dwc_b;     // kOut: [heads][d] or null
  UnitPlace at;           // Q, K, V and the gradients lie with the input strides, dO with the output strides
  BiasTables bt;          // with a bias only
};

struct AgentArgs {
  const void *X, *Y, *M1, *M2;      // in the element type
  const float *ts1, *ts2, *tw1, *rs1, *rs2, *rw1;      // as st1, st2, st3 and rs1, rs2, rw1 of TokenArgs
  const int* large;           // as in TokenArgs
  float *P1, *P2, *pm, *pl;
  int N, n, d, chunk, S;      // chunk: tokens per range (without a bias)
  float sc;
  UnitPlace at;               // Q, K, V lie with the input strides, dO with the output strides
  int gh, gw;
  // with a bias: ranges are `per` of the `pairs` pairs of columns (see bias_agent_kernel), a column being 16
  // neighbours in x of the seg_len image rows of one of `segs` segments
  int segs, seg_len, pairs, per;
  BiasTables bt;
  float *gt, *gr;             // parts of the gradients of T and R (null: not wanted), see BiasGradParts
  // the tokens' gradients of the kernels that take both sides (launch_both): kBc O1 = dQ, or Of where the pooling term is
  // still to come ([units][N][d]); kAgg O1 = dK, O2 = dV with the terms of G = dO as in TokenArgs
  void *O1, *O2;
  float* Of;
  float oscale;
  const void* G;
  float vk;
  const float* dwc_w;
};

// The kernels, compiled by backward_fused_kernels.hip (16-bit, no bias), backward_bias_{bf16,f16}.hip and
// backward_f32.hip.  dp: padded head width (16-bit 32 / 64 / 128, fp32 also 48 and 96); cols: 16-token columns per wave
// (token kernels) or 16-agent columns (agent kernels)
template <class E, bool BIAS>
hipError_t launch_token(int prob, int dp, int cols, const TokenArgs& a, dim3 grid, size_t lds, hipStream_t st);
template <class E, bool BIAS>
hipError_t launch_agent(int prob, int dp, int cols, const AgentArgs& a, dim3 grid, size_t lds, hipStream_t st);
// kBc / kAgg of units of at most 64 agents: the agents' and the tokens' gradients from one pass over the scores
template <class E, bool BIAS>
hipError_t launch_both(int prob, int dp, const AgentArgs& a, dim3 grid, size_t lds, hipStream_t st);

// --- backward_module.hip ---
// Fills the tables of the kinds in use ([0]: B2, [1]: B1; the same ld, a multiple of 64).
// Also clears `flags` (n_flags of them, may be null).
hipError_t launch_backward_bias_tables(const Problem& p, const BiasTables (&t)[2], const bool (&used)[2], int* flags, int n_flags,
                                       hipStream_t st);
// A flag that any number of lanes set
__device__ __forceinline__ void set_flag(int* f) { __hip_atomic_store(f, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Parts of one kind's bias gradients as the agent kernels leave them (fp32, unrounded score gradients):
//   gt [units][segs][cells][wp / 4][ld][4]    sums of (1 - f) dS and f dS over the image rows of a segment, for the
//                                             cell rows the segment touches (others are not written)
//   gr [units][xts][gh][ld]                   sums of dS over the 16 columns of an x-tile
// and sum, room for gt of one batch element and segment ([heads][cells][wp / 4][ld][4]).
struct BiasGradParts {
  const float *gt, *gr;
  float* sum;
  int segs, seg_len, cells, ld;
};
size_t dwc_param_part_floats(const Problem& p);
// The parameter gradients: the bias components' from parts ([0]: B2, [1]: B1; gt null: not in use), the convolution's
// from V and dO in the element type (d a multiple of 8, fp32 of 4, 16-byte rows); dwc_part: room for
// dwc_param_part_floats() floats.
hipError_t launch_backward_param_grads(const Problem& p, const BiasGradParts (&parts)[2], const BackwardParamGrads& pg,
                                       const void* V, const void* dO, float* dwc_part, hipStream_t st);

}  // namespace aa
