// Reference-quality HIP kernels for agent attention: every shape (d <= 256), every
// element type, plain fp32 VALU arithmetic.  They are the fp32 path and the safety
// net behind the MFMA kernels.  One wave works on one agent (aggregation) or one
// query token (broadcast); all waves of a block run the same trip counts so that
// block-wide barriers are always reached.
#include "kernels.h"

namespace aa {

constexpr int kWaves = 4;             // waves per block in aggregate / broadcast
constexpr int kMaxDPerLane = 4;       // d <= 64 * kMaxDPerLane


// ---------------------------------------------------------------------------
// A = Pooling(Q) (Sec. 4.2): block = one agent of one unit, thread = channel.
// ---------------------------------------------------------------------------
template <class E>
__global__ __launch_bounds__(64) void pool_generic_kernel(const typename E::T* __restrict__ Q,
                                                          typename E::T* __restrict__ A,
                                                          typename E::T* __restrict__ Alo, int N, int n, int d,
                                                          int heads, Layout lay, int gh, int gw, int ah, int aw) {
  const int a = blockIdx.x, u = blockIdx.y;
  const int ay = a / aw, ax = a % aw;
  const int y0 = pool_win_lo(ay, gh, ah), y1 = pool_win_hi(ay, gh, ah);
  const int x0 = pool_win_lo(ax, gw, aw), x1 = pool_win_hi(ax, gw, aw);
  const float inv = 1.0f / (float)((y1 - y0) * (x1 - x0));
  const typename E::T* q = Q + lay.in_unit(u, heads);
  for (int c = threadIdx.x; c < d; c += 64) {
    float acc = 0.0f;
    for (int y = y0; y < y1; ++y)
      for (int x = x0; x < x1; ++x) acc += E::to_f32(q[((size_t)y * lay.pitch(gw) + x) * lay.sn + c]);
    const float mean = acc * inv;
    const typename E::T hi = E::from_f32(mean);
    A[((size_t)u * n + a) * d + c] = hi;
    if (Alo) Alo[((size_t)u * n + a) * d + c] = E::from_f32(mean - E::to_f32(hi));      // what the rounding left over
  }
}

// ---------------------------------------------------------------------------
// The same for rows of whole 16-byte pieces and 16-byte aligned tensors: thread = one (agent, 16-byte piece) item, four
// window rows in flight.  grid = (ceil(pieces * n / 256), units).  Accumulation is fp32 in window order (row-major), as
// in the kernel above.
// ---------------------------------------------------------------------------
template <class E>
__global__ __launch_bounds__(256) void pool_chunk_kernel(const typename E::T* __restrict__ Q, typename E::T* __restrict__ A,
                                                         typename E::T* __restrict__ Alo, int N, int n, int d, int heads,
                                                         Layout lay, int gh, int gw, int ah, int aw) {
  using T = typename E::T;
  constexpr int PE = 16 / (int)sizeof(T);      // elements per piece
  struct alignas(16) Piece {
    T e[PE];
  };
  const int cpr = d / PE, u = blockIdx.y;
  const int item = blockIdx.x * 256 + threadIdx.x;
  if (item >= n * cpr) return;
  const int a = item / cpr, chunk = item - a * cpr;
  const int ay = a / aw, ax = a - ay * aw;
  const int y0 = pool_win_lo(ay, gh, ah), y1 = pool_win_hi(ay, gh, ah);
  const int x0 = pool_win_lo(ax, gw, aw), x1 = pool_win_hi(ax, gw, aw);
  const T* q = Q + lay.in_unit(u, heads) + PE * chunk;
  float acc[PE];
#pragma unroll
  for (int k = 0; k < PE; ++k) acc[k] = 0.0f;
  auto add = [&](const Piece& v) {
#pragma unroll
    for (int k = 0; k < PE; ++k) acc[k] += E::to_f32(v.e[k]);
  };
  for (int y = y0; y < y1; ++y) {
    const T* row = q + (size_t)y * lay.pitch(gw) * lay.sn;
    int x = x0;
    for (; x + 4 <= x1; x += 4) {
      Piece v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = *(const Piece*)(row + (size_t)(x + j) * lay.sn);
#pragma unroll
      for (int j = 0; j < 4; ++j) add(v[j]);
    }
    for (; x < x1; ++x) add(*(const Piece*)(row + (size_t)x * lay.sn));
  }
  const float inv = 1.0f / (float)((y1 - y0) * (x1 - x0));
  Piece w, wlo;
#pragma unroll
  for (int k = 0; k < PE; ++k) {
    const float mean = acc[k] * inv;
    w.e[k] = E::from_f32(mean);
    wlo.e[k] = E::from_f32(mean - E::to_f32(w.e[k]));      // what the rounding left over
  }
  *(Piece*)(A + ((size_t)u * n + a) * d + PE * chunk) = w;
  if (Alo) *(Piece*)(Alo + ((size_t)u * n + a) * d + PE * chunk) = wlo;
}

// ---------------------------------------------------------------------------
// Agent aggregation, split-N partial pass (Sec. 4.1 Eq. (3), bias of Eq. (5)).
// grid = (ceil(n / kWaves), S, units); wave w of a block owns agent 4*blockIdx.x + w
// and walks the tokens of split blockIdx.y in steps of 64 (one token per lane)
// with the running-maximum ("online") softmax.
// ---------------------------------------------------------------------------
template <class E>
__global__ __launch_bounds__(64 * kWaves) void aggregate_generic_kernel(
    const typename E::T* __restrict__ A, const typename E::T* __restrict__ Alo, const typename E::T* __restrict__ K,
    const typename E::T* __restrict__ V, BiasArgs b1, float scale, int N, int n, int d, int heads, Layout lay,
    int gh, int gw, int S, float* __restrict__ part_acc, float* __restrict__ part_m, float* __restrict__ part_l,
    float* __restrict__ VA_direct) {
  extern __shared__ float smem[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int a = blockIdx.x * kWaves + wave;
  const int s = blockIdx.y, u = blockIdx.z;
  const bool active = a < n;
  float* a_row = smem + wave * (d + 64);
  float* p_sh = a_row + d;

  const int chunk = (N + S - 1) / S;
  const int t0 = s * chunk;
  const int t1 = min(N, t0 + chunk);
  const typename E::T* Ku = K + lay.in_unit(u, heads);
  const typename E::T* Vu = V + lay.in_unit(u, heads);

  const int hd = u % heads;
  BiasArgs b = b1;
  if (b.col) b.col += (size_t)hd * n * gw;
  if (b.row) b.row += (size_t)hd * n * gh;
  if (b.blk) b.blk += (size_t)hd * n * b.h0 * b.w0;
  const bool has_bias = b.any();

  if (active)
    for (int c = lane; c < d; c += 64) {
      const size_t i = ((size_t)u * n + a) * d + c;
      a_row[c] = E::to_f32(A[i]) + (Alo ? E::to_f32(Alo[i]) : 0.0f);      // pooled agents come in two terms
    }
  __syncthreads();

  float m = -INFINITY, l = 0.0f;
  float acc[kMaxDPerLane] = {0.0f, 0.0f, 0.0f, 0.0f};

  for (int tb = t0; tb < t1; tb += 64) {
    const int t = tb + lane;
    const bool valid = active && t < t1;
    float sc = -INFINITY;
    if (valid) {
      const typename E::T* kr = Ku + lay.tok(t) * lay.sn;
      float dot = 0.0f;
#pragma unroll 8
      for (int c = 0; c < d; ++c) dot += a_row[c] * E::to_f32(kr[c]);
      sc = dot * scale;
      if (has_bias) sc += bias1_at(b, a, t / gw, t % gw, gh, gw);
    }
    const float m_new = fmaxf(m, wave_max(sc));
    const float p = valid ? __expf(sc - m_new) : 0.0f;
    const float alpha = active ? __expf(m - m_new) : 0.0f;   // m = -inf on the first step -> 0
    l = l * alpha + wave_sum(p);
    m = m_new;
    p_sh[lane] = p;
    __syncthreads();
    const int cnt = min(64, t1 - tb);
    if (active) {
#pragma unroll
      for (int k = 0; k < kMaxDPerLane; ++k) {
        const int c = lane + 64 * k;
        if (c < d) {
          float v = acc[k] * alpha;
#pragma unroll 8
          for (int j = 0; j < cnt; ++j) v += p_sh[j] * E::to_f32(Vu[lay.tok(tb + j) * lay.sn + c]);
          acc[k] = v;
        }
      }
    }
    __syncthreads();
  }

  if (active && VA_direct) {      // a single split is the whole sum: normalise here, as the merge would
    const float inv = 1.0f / l;
#pragma unroll
    for (int k = 0; k < kMaxDPerLane; ++k) {
      const int c = lane + 64 * k;
      if (c < d) VA_direct[((size_t)u * n + a) * d + c] = acc[k] * inv;
    }
  } else if (active) {
    const size_t row = ((size_t)u * S + s) * n + a;
#pragma unroll
    for (int k = 0; k < kMaxDPerLane; ++k) {
      const int c = lane + 64 * k;
      if (c < d) part_acc[row * d + c] = acc[k];
    }
    if (lane == 0) {
      part_m[row] = m;
      part_l[row] = l;
    }
  }
}

// ---------------------------------------------------------------------------
// Merge of the S split partials (log-sum-exp rule):
//   m = max_s m_s;  l = sum_s l_s e^{m_s-m};  VA = sum_s acc_s e^{m_s-m} / l.
// block = one agent of one unit; thread = channel.  Fixed summation order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void merge_generic_kernel(const float* __restrict__ part_acc,
                                                           const float* __restrict__ part_m,
                                                           const float* __restrict__ part_l, int S, int n, int d,
                                                           float* __restrict__ VA) {
  const int a = blockIdx.x, u = blockIdx.y;
  float m = -INFINITY;
  for (int s = 0; s < S; ++s) m = fmaxf(m, part_m[((size_t)u * S + s) * n + a]);
  float l = 0.0f;
  for (int s = 0; s < S; ++s) {
    const size_t row = ((size_t)u * S + s) * n + a;
    l += part_l[row] * __expf(part_m[row] - m);
  }
  const float inv = 1.0f / l;
  for (int c = threadIdx.x; c < d; c += 64) {
    float v = 0.0f;
    for (int s = 0; s < S; ++s) {
      const size_t row = ((size_t)u * S + s) * n + a;
      v += part_acc[row * d + c] * __expf(part_m[row] - m);
    }
    VA[((size_t)u * n + a) * d + c] = v * inv;
  }
}

// ---------------------------------------------------------------------------
// Agent broadcast (Eq. (3), bias B2 of Eq. (5)) with the module epilogue
// (+DWC(V) of Eq. (6), +k V of Appendix C.1).  grid = (ceil(N / kWaves), units);
// one wave per query token; scores over the n agents live in LDS.
// ---------------------------------------------------------------------------
template <class E>
__global__ __launch_bounds__(64 * kWaves) void broadcast_generic_kernel(
    const typename E::T* __restrict__ Q, const typename E::T* __restrict__ A, const typename E::T* __restrict__ Alo,
    const float* __restrict__ VA, const typename E::T* __restrict__ V, BiasArgs b2, const float* __restrict__ dwc_w,
    const float* __restrict__ dwc_b, float scale, float vk, int N, int n, int d, int heads, Layout lay, int gh,
    int gw, typename E::T* __restrict__ O) {
  extern __shared__ float smem[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * kWaves + wave;
  const int u = blockIdx.y;
  const bool active = i < N;
  float* q_row = smem + wave * (d + n);
  float* sc = q_row + d;

  const int hd = u % heads;
  BiasArgs b = b2;
  if (b.col) b.col += (size_t)hd * gw * n;
  if (b.row) b.row += (size_t)hd * gh * n;
  if (b.blk) b.blk += (size_t)hd * b.h0 * b.w0 * n;
  const bool has_bias = b.any();
  const int y = gw > 0 ? i / gw : 0, x = gw > 0 ? i % gw : 0;

  if (active)
    for (int c = lane; c < d; c += 64) q_row[c] = E::to_f32(Q[lay.in_unit(u, heads) + lay.tok(i) * lay.sn + c]);
  __syncthreads();

  float mx = -INFINITY;
  if (active)
    for (int a = lane; a < n; a += 64) {
      const typename E::T* ar = A + ((size_t)u * n + a) * d;
      float dot = 0.0f;
      if (Alo) {      // pooled agents come in two terms; block-uniform
        const typename E::T* al = Alo + ((size_t)u * n + a) * d;
#pragma unroll 8
        for (int c = 0; c < d; ++c) dot += q_row[c] * (E::to_f32(ar[c]) + E::to_f32(al[c]));
      } else {
#pragma unroll 8
        for (int c = 0; c < d; ++c) dot += q_row[c] * E::to_f32(ar[c]);
      }
      float s = dot * scale;
      if (has_bias) s += bias2_at(b, a, y, x, gh, gw, n);
      sc[a] = s;
      mx = fmaxf(mx, s);
    }
  mx = wave_max(mx);
  float sum = 0.0f;
  if (active)
    for (int a = lane; a < n; a += 64) {
      const float p = __expf(sc[a] - mx);
      sc[a] = p;
      sum += p;
    }
  sum = wave_sum(sum);
  __syncthreads();

  if (active) {
    const float inv = 1.0f / sum;
    const float* VAu = VA + (size_t)u * n * d;
    for (int c = lane; c < d; c += 64) {
      float o = 0.0f;
#pragma unroll 8
      for (int a = 0; a < n; ++a) o += sc[a] * VAu[(size_t)a * d + c];
      o *= inv;
      if (dwc_w) {
        const float* w9 = dwc_w + ((size_t)hd * d + c) * 9;
        float conv = dwc_b ? dwc_b[(size_t)hd * d + c] : 0.0f;
        for (int ky = -1; ky <= 1; ++ky)
          for (int kx = -1; kx <= 1; ++kx) {
            const int yy = y + ky, xx = x + kx;
            if (yy >= 0 && yy < gh && xx >= 0 && xx < gw)
              conv += w9[(ky + 1) * 3 + (kx + 1)] * E::to_f32(V[lay.in_unit(u, heads) + ((size_t)yy * lay.pitch(gw) + xx) * lay.sn + c]);
          }
        o += conv;
      }
      if (vk != 0.0f) o += vk * E::to_f32(V[lay.in_unit(u, heads) + lay.tok(i) * lay.sn + c]);
      O[lay.out_unit(u, heads) + lay.tok(i) * lay.on + c] = E::from_f32(o);
    }
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
#define AA_DISPATCH_DTYPE(dtype, ...)                  \
  switch (dtype) {                                     \
    case 0: { using E = ElemF32; __VA_ARGS__; } break;  \
    case 1: { using E = ElemF16; __VA_ARGS__; } break;  \
    case 2: { using E = ElemBF16; __VA_ARGS__; } break; \
    default: return hipErrorInvalidValue;              \
  }

// ---------------------------------------------------------------------------
// Agent bias evaluated once for all (agent, token) pairs of every head (Appendix B), in the padded
// layouts described at BiasArgs.  thread = one element.
// ---------------------------------------------------------------------------
// Entries of the tables are finite: a mask of the type's lowest value or of minus infinity is this, so that differences of
// two masked entries are zero and a row of them has a maximum.  Two of them are above what the MFMA kernels take for a
// maximum yet to be found (-1e30).  NaN stays NaN.
constexpr float kTableFloor = -2.5e29f;
__device__ __forceinline__ float floored(float v) { return v < kTableFloor ? kTableFloor : v; }

template <int KIND>
__device__ __forceinline__ void bias_dense_element(const BiasArgs& b, float* __restrict__ out, int n, int N,
                                                   int gh, int gw, unsigned i) {
  const unsigned NA = (unsigned)round_up64(n), NT = (unsigned)round_up64(N), q = i & 3;
  // kind 1: i = ((hd * NT/4 + t/4) * NA + a) * 4 + t%4, kind 2: i = ((hd * NA/4 + a/4) * N + t) * 4 + a%4
  const unsigned inner = KIND == 1 ? NA : (unsigned)N, rows = (KIND == 1 ? NT : NA) / 4;
  const unsigned row = (i >> 2) / inner, col = (i >> 2) - row * inner, hd = row / rows, quad = 4 * (row - hd * rows) + q;
  const int a = KIND == 1 ? (int)col : (int)quad, t = KIND == 1 ? (int)quad : (int)col;
  float v;
  const int y = t / gw, x = t - y * gw;
  if (t >= N || (KIND == 2 && a >= n)) {
    v = -INFINITY;
  } else if (a >= n) {
    v = 0.0f;
  } else {
    BiasArgs hb = b;
    if (KIND == 1) {
      if (hb.col) hb.col += (size_t)hd * n * gw;
      if (hb.row) hb.row += (size_t)hd * n * gh;
      if (hb.blk) hb.blk += (size_t)hd * n * hb.h0 * hb.w0;
      v = floored(kLog2e * bias1_at(hb, a, y, x, gh, gw));
    } else {
      if (hb.col) hb.col += (size_t)hd * gw * n;
      if (hb.row) hb.row += (size_t)hd * gh * n;
      if (hb.blk) hb.blk += (size_t)hd * hb.h0 * hb.w0 * n;
      v = floored(kLog2e * bias2_at(hb, a, y, x, gh, gw, n));
    }
  }
  out[i] = v;
}

// One launch for both kinds: the first blocks1 blocks fill the kind-1 table (when out1 is set), the rest the
// kind-2 table.
__global__ __launch_bounds__(256) void bias_dense_kernel(BiasArgs b1, float* __restrict__ out1, unsigned count1,
                                                         unsigned blocks1, BiasArgs b2, float* __restrict__ out2,
                                                         unsigned count2, int n, int N, int gh, int gw) {
  if (blockIdx.x < blocks1) {
    const unsigned i = blockIdx.x * 256u + threadIdx.x;
    if (i < count1) bias_dense_element<1>(b1, out1, n, N, gh, gw, i);
  } else {
    const unsigned i = (blockIdx.x - blocks1) * 256u + threadIdx.x;
    if (i < count2) bias_dense_element<2>(b2, out2, n, N, gh, gw, i);
  }
}

// ---------------------------------------------------------------------------
// The half-resized tables of BiasArgs (both kinds in one launch; a null output skips a kind).
// The tables are transposes of the parameters: the lanes lie along a table's contiguous direction (kind 1: agents, kind 2: columns
// or image rows), a wave stores 1 KB at a time, and reads the parameters in pieces of 16 bytes per lane, `quads` neighbouring ones,
// all asked for at once, for all cell rows a block makes.  What a cell row contributes comes from LDS, where the block
// component of the block's agents waits, `run` cell rows of it (kind 1 [agent][run w0], an odd stride apart; kind 2 [cell][16
// quads agents]); block grids too wide for that are read from memory.  Blocks: kind 1 64 agents x 16 quads columns (R: image
// rows), kind 2 64 columns (R: image rows) x 16 quads agents, a wave a quarter (of a narrow image more agents, so that no lane is idle).
// Bound by the way to the cold parameters and the stores behind it.  8 heads, 1024 agents, 128 x 128 tokens, 7 cell rows, all four
// tables (67 MB): 40.0 -> 19.9 us (one thread per 16 bytes of output and lanes in 8 x 8 tiles before: half of it was waiting for the
// parameters, which every thread gathered by itself); 8 of 80 x 100 tokens x 256 agents 9.9 -> 8.0.
// ---------------------------------------------------------------------------
// Block number = ((head * runs + run) * outer + o) * inner + i: blocks along the lanes (i) and along the waves' quads (o).  The
// inverses (see quotient) are 0 where they would not be exact.
struct HalfBlocks {
  unsigned count, inner, outer, runs;
  uint32_t inv_inner, inv_outer, inv_runs;
  __device__ __forceinline__ static unsigned div(unsigned v, unsigned by, uint32_t inverse) {
    return by == 1u ? v : inverse ? __umulhi(v, inverse) : v / by;
  }
  __device__ __forceinline__ void place(unsigned q, unsigned& i, unsigned& o, unsigned& run, unsigned& head) const {
    const unsigned t = div(q, inner, inv_inner), t2 = div(t, outer, inv_outer);
    i = q - t * inner, o = t - t2 * outer;
    head = div(t2, runs, inv_runs), run = t2 - head * runs;
  }
};
struct HalfKind {
  BiasArgs b;
  float *half, *rows;
  HalfBlocks cells, row_part;
  unsigned run;                                     // cell rows a block makes
  unsigned quads, row_quads;                        // 1, 2 or 4
  unsigned group_log2, row_group_log2;              // kind 2, images of up to 32 columns (rows): quads side by side in a wave
  unsigned staged, col_pieces, row_pieces;          // the block component goes through LDS; pieces of the others lie on 16 bytes
  uint32_t inv_per, inv_last;                       // quotient_inverse of run w0, and of what the last block has of it
};
typedef float table4 __attribute__((ext_vector_type(4)));
// `quads` neighbouring pieces of a parameter from p on, of which `valid` floats exist (the others: 0)
__device__ __forceinline__ void half_pieces(const float* p, int quads, int valid, bool pieces, table4 (&v)[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    v[m] = table4{0.f, 0.f, 0.f, 0.f};
    if (m >= quads || 4 * m >= valid) continue;
    if (pieces) {
      v[m] = *(const table4*)(p + 4 * m);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[m][j] = p[min(4 * m + j, valid - 1)];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (4 * m + j >= valid) v[m][j] = 0.f;
  }
}
template <int KIND>
__device__ __forceinline__ void half_block(const HalfKind& k, unsigned q, int n, int gw, unsigned NA, float* lds) {
  const BiasArgs& b = k.b;
  const int h0 = b.blk ? b.h0 : 1, w0 = b.blk ? b.w0 : 1, Q = (int)k.quads, span = (int)(16 * Q) << k.group_log2;
  const int lane = (threadIdx.x & 63) & (63 >> k.group_log2);      // narrow images: several of a wave's quads side by side
  const int w = (int)((threadIdx.x >> 6 << k.group_log2) + ((threadIdx.x & 63) >> (6 - k.group_log2)));
  unsigned li, wi, c0, hd;
  k.cells.place(q, li, wi, c0, hd);
  c0 *= k.run;
  const int cells = min((int)k.run, h0 - (int)c0);
  const int a = KIND == 1 ? (int)(64 * li) + lane : (int)wi * span + 4 * Q * w;      // this thread's agent, or the first of its agents
  const int x = KIND == 1 ? (int)wi * span + 4 * Q * w : (int)(64 * li) + lane;      // its first column, or its column
  table4 col[4];
  const int valid = !b.col || a >= n || x >= gw ? 0 : KIND == 1 ? gw - x : n - a;
  half_pieces(b.col + (KIND == 1 ? ((size_t)hd * n + a) * gw + x : ((size_t)hd * gw + x) * n + a), Q, valid, k.col_pieces, col);
  const int stride = KIND == 1 ? (int)(k.run * (unsigned)w0) | 1 : span;      // of an agent's part, of a cell's
  if (b.blk && k.staged) {      // four loads in flight; floored here, once
    const int per = cells * w0, count = (KIND == 1 ? 64 : span) * per;
    const uint32_t inv = cells == (int)k.run ? k.inv_per : k.inv_last;
    const int shift = 31 - __clz(span);
    for (int i0 = threadIdx.x; i0 < count; i0 += 4 * 256) {
      float v[4];
      int at[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int i = min(i0 + 256 * m, count - 1), ai = KIND == 1 ? quotient(i, inv) : i & (span - 1), e = KIND == 1 ? i - ai * per : i >> shift;
        const int ag = (KIND == 1 ? (int)(64 * li) : (int)wi * span) + ai, agc = min(ag, n - 1);
        v[m] = KIND == 1 ? b.blk[((size_t)hd * n + agc) * h0 * w0 + (size_t)c0 * w0 + e] : b.blk[(((size_t)hd * h0 + c0) * w0 + e) * n + agc];
        v[m] = ag < n ? v[m] : 0.f;
        at[m] = KIND == 1 ? ai * stride + e : i;
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) lds[at[m]] = floored(v[m]);
    }
    __syncthreads();
  }
  if (KIND == 2 && x >= gw) return;
  int x0[4], x1[4];
  float fx[4];
  if (KIND == 2) bilinear_coord(x, gw, w0, x0[0], x1[0], fx[0]);
  const size_t cell_floats = (size_t)gw * NA;
  for (int m = 0; m < Q; ++m) {
    const int am = KIND == 1 ? a : a + 4 * m, xm = KIND == 1 ? x + 4 * m : x;
    if (KIND == 1 ? xm >= gw : am >= (int)NA) return;
    if (KIND == 1) {
#pragma unroll
      for (int j = 0; j < 4; ++j) bilinear_coord(min(xm + j, gw - 1), gw, w0, x0[j], x1[j], fx[j]);
    }
    const table4 cv = m == 0 ? col[0] : m == 1 ? col[1] : m == 2 ? col[2] : col[3];
    float* to = k.half + ((size_t)hd * h0 + c0) * cell_floats +
                (KIND == 1 ? ((size_t)(xm >> 2) * NA + am) * 4 : ((size_t)(am >> 2) * gw + xm) * 4);
    const float* part = lds + (KIND == 1 ? lane * stride : 4 * Q * w + 4 * m);
    for (int c = 0; c < cells; ++c, to += cell_floats) {
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float p0 = 0.f, p1 = 0.f;
        const int xa = KIND == 1 ? x0[j] : x0[0], xb = KIND == 1 ? x1[j] : x1[0];
        if (b.blk && k.staged) {
          if (KIND == 1) p0 = part[c * w0 + xa], p1 = part[c * w0 + xb];
          else p0 = part[(c * w0 + xa) * stride + j], p1 = part[(c * w0 + xb) * stride + j];
        } else if (b.blk && (KIND == 1 ? am : am + j) < n) {
          const float* p = KIND == 1 ? b.blk + (((size_t)hd * n + am) * h0 + c0 + c) * w0 : b.blk + ((size_t)hd * h0 + c0 + c) * w0 * n + am + j;
          p0 = floored(KIND == 1 ? p[xa] : p[(size_t)xa * n]), p1 = floored(KIND == 1 ? p[xb] : p[(size_t)xb * n]);
        }
        v[j] = floored((cv[j] + (p0 + (p1 - p0) * (KIND == 1 ? fx[j] : fx[0]))) * kLog2e);
      }
      *(table4*)to = table4{v[0], v[1], v[2], v[3]};
    }
  }
}
template <int KIND>
__device__ __forceinline__ void half_row_block(const HalfKind& k, unsigned q, int n, int gh, unsigned NA) {
  const BiasArgs& b = k.b;
  const int Q = (int)k.row_quads, span = (int)(16 * Q) << k.row_group_log2, lane = (threadIdx.x & 63) & (63 >> k.row_group_log2);
  const int w = (int)((threadIdx.x >> 6 << k.row_group_log2) + ((threadIdx.x & 63) >> (6 - k.row_group_log2)));
  unsigned li, wi, run, hd;
  k.row_part.place(q, li, wi, run, hd);
  const int a = KIND == 1 ? (int)(64 * li) + lane : (int)wi * span + 4 * Q * w;
  const int y = KIND == 1 ? (int)wi * span + 4 * Q * w : (int)(64 * li) + lane;
  table4 v[4];
  const int valid = a >= n || y >= gh ? 0 : KIND == 1 ? gh - y : n - a;
  half_pieces(b.row + (KIND == 1 ? ((size_t)hd * n + a) * gh + y : ((size_t)hd * gh + y) * n + a), Q, valid, k.row_pieces, v);
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    if (m >= Q) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[m][j] = floored(v[m][j] * kLog2e);
    if (KIND == 1) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (y + 4 * m + j < gh) k.rows[((size_t)hd * gh + y + 4 * m + j) * NA + a] = v[m][j];
    } else if (y < gh && a + 4 * m < (int)NA) {
      *(table4*)(k.rows + (((size_t)hd * (NA >> 2) + (a >> 2) + m) * gh + y) * 4) = v[m];
    }
  }
}
__global__ __launch_bounds__(256) void bias_half_kernel(HalfKind k1, HalfKind k2, int n, int gh, int gw) {
  extern __shared__ __align__(16) float half_lds[];
  const unsigned NA = (unsigned)round_up64(n);
  unsigned q = blockIdx.x;
  if (q < k1.cells.count) return half_block<1>(k1, q, n, gw, NA, half_lds);
  q -= k1.cells.count;
  if (q < k2.cells.count) return half_block<2>(k2, q, n, gw, NA, half_lds);
  q -= k2.cells.count;
  if (q < k1.row_part.count) return half_row_block<1>(k1, q, n, gh, NA);
  half_row_block<2>(k2, q - k1.row_part.count, n, gh, NA);
}

size_t bias_half_floats(int heads, int n, int gw, int he) { return (size_t)heads * round_up64(n) * he * gw; }
size_t bias_rows_floats(int heads, int n, int gh) { return (size_t)heads * round_up64(n) * gh; }

hipError_t launch_bias_half(const Problem& p, float* half1, float* rows1, float* half2, float* rows2, hipStream_t st) {
  // the caller keeps every table below 2 GiB, so 32-bit counts suffice
  const unsigned NA = (unsigned)round_up64(p.n), H = (unsigned)p.heads;
  constexpr int kStageFloats = 8192;
  int lds = 0;
  auto kind = [&](const BiasArgs& b, float* half, float* rows, bool first) {
    HalfKind k{};
    k.b = b, k.half = half, k.rows = rows;
    const int h0 = b.blk ? b.h0 : 1, w0 = b.blk ? b.w0 : 1;
    auto group = [&](int length) {
      unsigned g = 0;
      while (!first && (length << (g + 1)) <= 64 && 16u << (g + 1) <= NA) ++g;
      return g;
    };
    k.group_log2 = group(p.gw), k.row_group_log2 = group(p.gh);
    auto blocks = [&](int length, unsigned quads, unsigned runs) {      // along `length` columns or image rows
      const unsigned span = (16 * quads) << group(length);
      HalfBlocks n{0, first ? NA >> 6 : ((unsigned)length + 63) >> 6, ((first ? (unsigned)length : NA) + span - 1) / span, runs, 0, 0, 0};
      n.count = H * n.inner * n.outer * runs;
      auto inverse = [&](unsigned by) { return (unsigned long long)n.count * by >> 32 == 0 ? quotient_inverse((int)by) : 0u; };
      n.inv_inner = inverse(n.inner), n.inv_outer = inverse(n.outer), n.inv_runs = inverse(runs);
      return n;
    };
    // The widest pieces that leave two blocks a CU, and as many cell rows a block as leave one and fit LDS.  Kernel alone in us, one
    // block for the pieces / this / four, and this with two blocks a CU left by the cell rows; 7 cell rows: 8 heads of 128 x 128
    // tokens x 1024 agents 19.8 / 19.9 / 20.2, 23.8; 8 of 80 x 100 x 256 12.7 / 8.0 / 7.6, 12.1; 4 of 96 x 96 x 576 13.4 / 8.7 / 8.0,
    // 12.2; 8 of 17 x 40 x 160 6.5 / 5.1 / 5.1, 5.6; 8 of 128 x 4 x 66 4.1 / 4.2 / 4.8, 4.1.
    auto widest = [&](int length, int cell_rows) {
      unsigned quads = 4;
      while (quads > 1 && blocks(length, quads, cell_rows).count < 2u * kComputeUnits) quads /= 2;
      return quads;
    };
    k.quads = widest(p.gw, h0), k.row_quads = widest(p.gh, 1);
    auto floats = [&](int run) { return first ? 64 * ((run * w0) | 1) : ((16 * (int)k.quads) << k.group_log2) * run * w0; };
    int run = std::max(1, std::min(h0, (int)(blocks(p.gw, k.quads, h0).count / (unsigned)kComputeUnits)));
    while (run > 1 && floats(run) > kStageFloats) --run;
    const int runs = (h0 + run - 1) / run;
    k.run = (unsigned)run;
    k.staged = b.blk && run > 1 && floats(run) <= kStageFloats;      // (a single one is asked for beside the column component)
    k.inv_per = quotient_inverse(run * w0), k.inv_last = quotient_inverse((h0 - (runs - 1) * run) * w0);
    auto pieces = [&](const float* from, int length) { return ((uintptr_t)from % 16 == 0 && (first ? length : p.n) % 4 == 0) ? 1u : 0u; };
    k.col_pieces = pieces(b.col, p.gw), k.row_pieces = pieces(b.row, p.gh);
    if (half) {
      k.cells = blocks(p.gw, k.quads, runs);
      if (k.staged) lds = std::max(lds, floats(run) * 4);
    }
    if (rows) k.row_part = blocks(p.gh, k.row_quads, 1);
    return k;
  };
  const HalfKind k1 = kind(p.b1, half1, rows1, true), k2 = kind(p.b2, half2, rows2, false);
  const unsigned total = k1.cells.count + k2.cells.count + k1.row_part.count + k2.row_part.count;
  if (total == 0) return hipSuccess;
  bias_half_kernel<<<dim3(total), dim3(256), (size_t)lds, st>>>(k1, k2, p.n, p.gh, p.gw);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Matrix form of B1's block component (see BiasArgs::wt / blkop): one thread per 16 bytes (eight fp16 values).
// Segments: the token weights [N][64], then the block operand [heads][n_pad][64] (times log2 e).
// ---------------------------------------------------------------------------
constexpr int kBiasK = 64;      // k-slots of the matrix form
__device__ __forceinline__ uint16_t f16_bits(float v) {
  const _Float16 h = (_Float16)v;
  return __builtin_bit_cast(uint16_t, h);
}
__global__ __launch_bounds__(256) void bias_matrix_kernel(uint16_t* __restrict__ wt, uint16_t* __restrict__ k1, BiasArgs b1,
                                                          int n, int gh, int gw, unsigned q_wt, unsigned q_k) {
  unsigned q = blockIdx.x * 256u + threadIdx.x;
  const bool weights = q < q_wt;
  if (!weights) {
    q -= q_wt;
    if (q >= q_k) return;
  }
  const unsigned piece = q & 7u, row = q >> 3;
  const int h0 = b1.h0, w0 = b1.w0;
  uint16_t out[8];
  if (weights) {      // row = token
    const int y = (int)row / gw, x = (int)row - y * gw;
    int i0, i1, j0, j1;
    float fy, fx;
    bilinear_coord(y, gh, h0, i0, i1, fy);
    bilinear_coord(x, gw, w0, j0, j1, fx);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 8 * (int)piece + e, i = k / w0, j = k - i * w0;
      float v = 0.0f;
      if (k < h0 * w0) {
        const float wy = (i == i0 ? 1.0f - fy : 0.0f) + (i == i1 ? fy : 0.0f);
        const float wx = (j == j0 ? 1.0f - fx : 0.0f) + (j == j1 ? fx : 0.0f);
        v = wy * wx;
      }
      out[e] = f16_bits(v);
    }
  } else {            // row = (head, padded agent)
    const unsigned NA = (unsigned)round_up64(n), a = row % NA, hd = row / NA;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 8 * (int)piece + e;
      float v = 0.0f;
      if ((int)a < n && k < h0 * w0) v = b1.blk[((size_t)hd * n + a) * h0 * w0 + k];
      v *= kLog2e;      // within fp16: a mask past its range would meet the zero weights of other tokens as an infinity
      out[e] = f16_bits(v < -65504.0f ? -65504.0f : v > 65504.0f ? 65504.0f : v);
    }
  }
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  *(u32x4*)((weights ? wt : k1) + (size_t)row * kBiasK + 8 * piece) =
      u32x4{(uint32_t)out[0] | ((uint32_t)out[1] << 16), (uint32_t)out[2] | ((uint32_t)out[3] << 16),
            (uint32_t)out[4] | ((uint32_t)out[5] << 16), (uint32_t)out[6] | ((uint32_t)out[7] << 16)};
}

size_t bias_wt_bytes(int N) { return (size_t)N * kBiasK * 2; }
size_t bias_blkop_bytes(int heads, int n) { return (size_t)heads * round_up64(n) * kBiasK * 2; }

hipError_t launch_bias_matrix(const Problem& p, uint16_t* wt, uint16_t* k1, hipStream_t st) {
  if (!wt || !k1) return hipSuccess;
  const unsigned q_wt = (unsigned)p.N * 8u, q_k = (unsigned)p.heads * (unsigned)round_up64(p.n) * 8u;
  const size_t total = (size_t)q_wt + q_k;
  bias_matrix_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st>>>(wt, k1, p.b1, p.n, p.gh, p.gw, q_wt, q_k);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Dense <-> strided copies of a [units][N][d] token tensor (the backward pass works on dense copies of
// strided tensors; the forward pass on dense copies of the windows of an image when the kernel family that
// serves the shape does not address windows in place).  T only carries the size of what a thread moves:
// one element, or a 16-byte piece of 8 16-bit elements (d and every stride a multiple of 8 then).
// ---------------------------------------------------------------------------
typedef uint32_t piece16_t __attribute__((ext_vector_type(4)));

template <class T, int EPT, bool TO_DENSE>
__global__ __launch_bounds__(256) void restride_kernel(const T* __restrict__ src, T* __restrict__ dst, int N, int d,
                                                       int heads, Layout lay, bool out_layout, size_t count) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  const int dp = d / EPT;                      // pieces per row
  const int c = (int)(i % dp);
  const size_t row = i / dp;
  const int t = (int)(row % N), u = (int)(row / N);
  const size_t strided_elems = out_layout ? lay.out_unit(u, heads) + lay.tok(t) * lay.on
                                          : lay.in_unit(u, heads) + lay.tok(t) * lay.sn;
  const size_t strided = strided_elems / EPT + c;
  if (TO_DENSE)
    dst[i] = src[strided];
  else
    dst[strided] = src[i];
}

hipError_t launch_restride(const Problem& p, bool to_dense, bool out_layout, const void* src, void* dst, hipStream_t st) {
  const Layout& L = p.lay;
  const bool wide = p.dtype != 0 && p.d % 8 == 0 && L.sb % 8 == 0 && L.sh % 8 == 0 && L.sn % 8 == 0 && L.ob % 8 == 0 &&
                    L.oh % 8 == 0 && L.on % 8 == 0 && ((uintptr_t)src & 15) == 0 && ((uintptr_t)dst & 15) == 0;
  const size_t count = (size_t)p.units * p.N * p.d / (wide ? 8 : 1);
  const dim3 grid((unsigned)((count + 255) / 256));
#define AA_RESTRIDE(T, EPT)                                                                                              \
  do {                                                                                                                   \
    if (to_dense)                                                                                                        \
      restride_kernel<T, EPT, true><<<grid, dim3(256), 0, st>>>((const T*)src, (T*)dst, p.N, p.d, p.heads, L, out_layout, count); \
    else                                                                                                                 \
      restride_kernel<T, EPT, false><<<grid, dim3(256), 0, st>>>((const T*)src, (T*)dst, p.N, p.d, p.heads, L, out_layout, count); \
  } while (0)
  if (p.dtype == 0) AA_RESTRIDE(float, 1);
  else if (wide) AA_RESTRIDE(piece16_t, 8);
  else AA_RESTRIDE(uint16_t, 1);
#undef AA_RESTRIDE
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Bias of a linear projection: Y[r][c] += bias[c].  thread = one element.
// ---------------------------------------------------------------------------
template <class E>
__global__ __launch_bounds__(256) void add_row_bias_kernel(typename E::T* __restrict__ Y, const typename E::T* __restrict__ bias,
                                                           size_t count, int cols) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  Y[i] = E::from_f32(E::to_f32(Y[i]) + E::to_f32(bias[i % cols]));
}

hipError_t launch_add_row_bias(int dtype, void* Y, const void* bias, size_t rows, int cols, hipStream_t st) {
  const size_t count = rows * (size_t)cols;
  const dim3 grid((unsigned)((count + 255) / 256));
  AA_DISPATCH_DTYPE(dtype, add_row_bias_kernel<E><<<grid, dim3(256), 0, st>>>((typename E::T*)Y, (const typename E::T*)bias, count, cols));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Bias component adapted to another agent grid (Appendix D.1 / D.2, "Numbers of agent tokens"): the tensor is
// viewed as [outer][ah][aw][inner] and every [ah][aw] image is bilinearly interpolated (half-pixel centres, as
// for the block bias) to [ah2][aw2].  thread = one output element.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void resize_agent_axis_kernel(const float* __restrict__ src, float* __restrict__ dst,
                                                                int ah, int aw, int inner, int ah2, int aw2,
                                                                size_t count) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  const int c = (int)(i % inner);
  const size_t t = i / inner;
  const int ax = (int)(t % aw2), ay = (int)((t / aw2) % ah2);
  const size_t o = t / ((size_t)aw2 * ah2);
  int y0, y1, x0, x1;
  float fy, fx;
  bilinear_coord(ay, ah2, ah, y0, y1, fy);
  bilinear_coord(ax, aw2, aw, x0, x1, fx);
  const float* p = src + o * ah * aw * inner + c;
  const float v00 = p[(size_t)(y0 * aw + x0) * inner], v01 = p[(size_t)(y0 * aw + x1) * inner];
  const float v10 = p[(size_t)(y1 * aw + x0) * inner], v11 = p[(size_t)(y1 * aw + x1) * inner];
  const float top = v00 + (v01 - v00) * fx, bot = v10 + (v11 - v10) * fx;
  dst[i] = top + (bot - top) * fy;
}

hipError_t launch_resize_agent_axis(const float* src, float* dst, size_t outer, int ah, int aw, int inner, int ah2,
                                    int aw2, hipStream_t st) {
  const size_t count = outer * ah2 * aw2 * inner;
  if (count == 0) return hipSuccess;
  resize_agent_axis_kernel<<<dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st>>>(src, dst, ah, aw, inner, ah2, aw2,
                                                                                      count);
  return hipGetLastError();
}

size_t bias_dense_floats(int kind, int heads, int n, int N) {
  return kind == 1 ? (size_t)heads * round_up64(n) * round_up64(N) : (size_t)heads * N * round_up64(n);
}

hipError_t launch_bias_dense(const Problem& p, float* out1, float* out2, hipStream_t st) {
  // (the caller keeps a table below 2 GiB)
  const unsigned count1 = out1 ? (unsigned)bias_dense_floats(1, p.heads, p.n, p.N) : 0;
  const unsigned count2 = out2 ? (unsigned)bias_dense_floats(2, p.heads, p.n, p.N) : 0;
  const unsigned blocks1 = (count1 + 255) / 256, blocks2 = (count2 + 255) / 256;
  if (blocks1 + blocks2 == 0) return hipSuccess;
  bias_dense_kernel<<<dim3(blocks1 + blocks2), dim3(256), 0, st>>>(p.b1, out1, count1, blocks1, p.b2, out2, count2, p.n, p.N,
                                                                   p.gh, p.gw);
  return hipGetLastError();
}

hipError_t launch_pool_generic(const Problem& p, const void* Q, void* A, void* Alo, hipStream_t st) {
  dim3 grid(p.n, p.units);
  if (p.dtype == 0) Alo = nullptr;      // fp32 agents carry no residual worth keeping
  AA_DISPATCH_DTYPE(p.dtype, pool_generic_kernel<E><<<grid, dim3(64), 0, st>>>(
      (const typename E::T*)Q, (typename E::T*)A, (typename E::T*)Alo, p.N, p.n, p.d, p.heads, p.lay, p.gh, p.gw, p.ah, p.aw));
  return hipGetLastError();
}

hipError_t launch_pool_chunk(const Problem& p, const void* Q, void* A, void* Alo, hipStream_t st) {
  const dim3 grid((p.n * (p.d / (p.dtype == 0 ? 4 : 8)) + 255) / 256, p.units);
  if (p.dtype == 0) Alo = nullptr;      // fp32 agents carry no residual worth keeping
  AA_DISPATCH_DTYPE(p.dtype, pool_chunk_kernel<E><<<grid, dim3(256), 0, st>>>(
      (const typename E::T*)Q, (typename E::T*)A, (typename E::T*)Alo, p.N, p.n, p.d, p.heads, p.lay, p.gh, p.gw, p.ah, p.aw));
  return hipGetLastError();
}

// VA_direct: with one split (part.S == 1) the kernel may write the normalised V_A itself (no merge launch)
hipError_t launch_aggregate_generic(const Problem& p, const void* A, const void* Alo, const void* K, const void* V,
                                    const Partials& part, float* VA_direct, hipStream_t st) {
  dim3 grid((p.n + kWaves - 1) / kWaves, part.S, p.units);
  const size_t lds = (size_t)kWaves * (p.d + 64) * sizeof(float);
  AA_DISPATCH_DTYPE(p.dtype, aggregate_generic_kernel<E><<<grid, dim3(64 * kWaves), lds, st>>>(
      (const typename E::T*)A, (const typename E::T*)Alo, (const typename E::T*)K, (const typename E::T*)V, p.b1,
      p.scale1, p.N, p.n, p.d,
      p.heads, p.lay, p.gh, p.gw, part.S, part.acc, part.m, part.l, part.S == 1 ? VA_direct : nullptr));
  return hipGetLastError();
}

hipError_t launch_merge_generic(const Problem& p, const Partials& part, float* VA, hipStream_t st) {
  dim3 grid(p.n, p.units);
  merge_generic_kernel<<<grid, dim3(64), 0, st>>>(part.acc, part.m, part.l, part.S, p.n, p.d, VA);
  return hipGetLastError();
}

size_t broadcast_generic_lds_bytes(int n, int d) { return (size_t)kWaves * (n + d) * sizeof(float); }

hipError_t launch_broadcast_generic(const Problem& p, const void* Q, const void* A, const void* Alo, const float* VA,
                                    const void* V, void* out, hipStream_t st) {
  dim3 grid((p.N + kWaves - 1) / kWaves, p.units);
  const size_t lds = broadcast_generic_lds_bytes(p.n, p.d);
  AA_DISPATCH_DTYPE(p.dtype, broadcast_generic_kernel<E><<<grid, dim3(64 * kWaves), lds, st>>>(
      (const typename E::T*)Q, (const typename E::T*)A, (const typename E::T*)Alo, VA, (const typename E::T*)V, p.b2, p.dwc_w, p.dwc_b,
      p.scale2, p.vk, p.N, p.n, p.d, p.heads, p.lay, p.gh, p.gw, (typename E::T*)out));
  return hipGetLastError();
}

}  // namespace aa
