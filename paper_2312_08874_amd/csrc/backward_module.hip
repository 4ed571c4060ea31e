// Module terms of the recomputing backward: the agent-bias tables its kernels read, the sums of the bias gradients
// they leave behind, and the depthwise convolution's parameter gradients.  No atomics, every sum in a fixed order.
#include "backward_fused.h"
#include "mfma_common.h"

namespace aa {

namespace {

// ---------------------------------------------------------------------------
// Tables of one bias kind (BiasTables).  Blocks [0, tblocks): a thread takes four columns x four agents of one cell
// row, lanes along the agents (tx is then written in one piece per wave, ta in 64-byte pieces).  The next rblocks: R,
// four agents per thread.  The rest: the image rows' interpolation along y.
// ---------------------------------------------------------------------------
template <int KIND>
__global__ __launch_bounds__(256) void bias_tables_kernel(BiasArgs b, float* __restrict__ ta, float* __restrict__ tx,
                                                          float* __restrict__ rows, YInfo* __restrict__ yi, int heads, int n,
                                                          int gh, int gw, int cells, int ld, unsigned tblocks, unsigned rblocks) {
  const int l4 = ld / 4, wp = (gw + 15) / 16 * 16;
  if (blockIdx.x < tblocks) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int a4 = (int)(i % l4);
    const size_t rest = i / l4;
    const int x4 = (int)(rest % (wp / 4));
    const int cell = (int)(rest / (wp / 4) % cells), hd = (int)(rest / (wp / 4) / cells);
    if (hd >= heads) return;
    float v[4][4];      // [column][agent]
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int x = 4 * x4 + j;
      int x0 = 0, x1 = 0;
      float fx = 0.0f;
      if (b.blk) bilinear_coord(min(x, gw - 1), gw, b.w0, x0, x1, fx);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int a = 4 * a4 + k;
        float s = 0.0f;
        if (x >= gw) {
          s = -1.0e30f;      // a column past the image weighs nothing
        } else if (a < n) {
          if (b.col) s = KIND == 1 ? b.col[((size_t)hd * n + a) * gw + x] : b.col[((size_t)hd * gw + x) * n + a];
          if (b.blk) {
            const size_t step = KIND == 1 ? 1 : n;
            const float* q = KIND == 1 ? b.blk + (((size_t)hd * n + a) * b.h0 + cell) * b.w0
                                       : b.blk + ((size_t)hd * b.h0 + cell) * b.w0 * n + a;
            const float v0 = q[x0 * step], v1 = q[x1 * step];
            s += v0 + (v1 - v0) * fx;
          }
          s *= kLog2e;
        }
        v[j][k] = s;
      }
    }
    const size_t base = ((size_t)hd * cells + cell) * ld * wp;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<f32x4*>(ta + base + ((size_t)a4 * wp + 4 * x4 + j) * 4) = f32x4{v[j][0], v[j][1], v[j][2], v[j][3]};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      *reinterpret_cast<f32x4*>(tx + base + ((size_t)x4 * ld + 4 * a4 + k) * 4) = f32x4{v[0][k], v[1][k], v[2][k], v[3][k]};
  } else if (blockIdx.x < tblocks + rblocks) {
    const size_t i = (size_t)(blockIdx.x - tblocks) * 256 + threadIdx.x;
    const int a4 = (int)(i % l4), y = (int)(i / l4 % gh), hd = (int)(i / l4 / gh);
    if (hd >= heads) return;
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int a = 4 * a4 + k;
      v[k] = a < n ? kLog2e * (KIND == 1 ? b.row[((size_t)hd * n + a) * gh + y] : b.row[((size_t)hd * gh + y) * n + a]) : 0.0f;
    }
    *reinterpret_cast<f32x4*>(rows + ((size_t)hd * gh + y) * ld + 4 * a4) = f32x4{v[0], v[1], v[2], v[3]};
  } else {
    const int y = (int)(blockIdx.x - tblocks - rblocks) * 256 + threadIdx.x;
    if (y >= gh) return;
    int i0, i1;
    float f;
    bilinear_coord(y, gh, cells, i0, i1, f);
    int next = y + 1;
    for (; next < gh; ++next) {
      int c;
      float g;
      bilinear_coord(next, gh, cells, c, i1, g);
      if (c != i0) break;
    }
    yi[y] = YInfo{i0, next, i0 >= cells - 1 ? 0.0f : f, 0};
  }
}

// cell rows [c0, c1] that the image rows of segment s touch
__device__ __forceinline__ void segment_cells(int s, int seg_len, int gh, int cells, int& c0, int& c1) {
  int up;
  float f;
  bilinear_coord(s * seg_len, gh, cells, c0, up, f);
  bilinear_coord(min(gh, (s + 1) * seg_len) - 1, gh, cells, c1, up, f);
  c1 = min(c1 + 1, cells - 1);
}

// sum [heads][cells][wp / 4][ld] of four columns each: the parts of the batch's units and their segments, in order
__global__ __launch_bounds__(256) void bias_grad_sum_kernel(const f32x4* __restrict__ gt, f32x4* __restrict__ sum, int batch,
                                                            int heads, int segs, int seg_len, int gh, int cells, size_t per_cell) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)heads * cells * per_cell) return;
  const size_t e = i % per_cell;
  const int cell = (int)(i / per_cell % cells), hd = (int)(i / per_cell / cells);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < segs; ++s) {
    int c0, c1;
    segment_cells(s, seg_len, gh, cells, c0, c1);
    if (cell < c0 || cell > c1) continue;
    const f32x4* p = gt + (((size_t)hd * segs + s) * cells + cell) * per_cell + e;
    const size_t step = (size_t)heads * segs * cells * per_cell;
#pragma unroll 4
    for (int bt = 0; bt < batch; ++bt) acc += p[bt * step];
  }
  sum[i] = acc;
}

// The components' gradients from the sums: column blocks, then row blocks, then block-cell blocks, one output element
// per thread, lanes along the agents.  live = 0: the softmax has a single entry, is constant, and its scores' gradients
// are zero (the parts hold the rounding error of a difference of equal terms).
template <int KIND>
__global__ __launch_bounds__(256) void bias_grad_out_kernel(const f32x4* __restrict__ sum, const float* __restrict__ gr,
                                                            float* __restrict__ col, float* __restrict__ row,
                                                            float* __restrict__ blk, int batch, int heads, int n, int gh, int gw,
                                                            int cells, int w0, int ld, float live, unsigned cblocks,
                                                            unsigned rblocks) {
  const int xts = (gw + 15) / 16, wp = 16 * xts;
  const size_t per_cell = (size_t)wp / 4 * ld;
  if (blockIdx.x < cblocks) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int a = (int)(i % n), x = (int)(i / n % gw), hd = (int)(i / n / gw);
    if (hd >= heads) return;
    float v = 0.0f;
    for (int c = 0; c < cells; ++c) v += sum[((size_t)hd * cells + c) * per_cell + (size_t)(x >> 2) * ld + a][x & 3];
    col[KIND == 1 ? ((size_t)hd * n + a) * gw + x : ((size_t)hd * gw + x) * n + a] = live * v;
  } else if (blockIdx.x < cblocks + rblocks) {
    const size_t i = (size_t)(blockIdx.x - cblocks) * 256 + threadIdx.x;
    const int a = (int)(i % n), y = (int)(i / n % gh), hd = (int)(i / n / gh);
    if (hd >= heads) return;
    float v = 0.0f;
    for (int bt = 0; bt < batch; ++bt)
#pragma unroll 4
      for (int t = 0; t < xts; ++t) v += gr[((((size_t)bt * heads + hd) * xts + t) * gh + y) * ld + a];
    row[KIND == 1 ? ((size_t)hd * n + a) * gh + y : ((size_t)hd * gh + y) * n + a] = live * v;
  } else {
    const size_t i = (size_t)(blockIdx.x - cblocks - rblocks) * 256 + threadIdx.x;
    const int a = (int)(i % n), q = (int)(i / n % w0), cell = (int)(i / n / w0 % cells), hd = (int)(i / n / w0 / cells);
    if (hd >= heads) return;
    float v = 0.0f;
    for (int x4 = 0; 4 * x4 < gw; ++x4) {
      float wx[4];
      bool any = false;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        int x0, x1;
        float fx;
        bilinear_coord(min(4 * x4 + j, gw - 1), gw, w0, x0, x1, fx);
        wx[j] = 4 * x4 + j < gw ? (x0 == q ? 1.0f - fx : 0.0f) + (x1 == q ? fx : 0.0f) : 0.0f;
        any = any || wx[j] != 0.0f;
      }
      if (!any) continue;
      const f32x4 s = sum[((size_t)hd * cells + cell) * per_cell + (size_t)x4 * ld + a];
#pragma unroll
      for (int j = 0; j < 4; ++j) v = fmaf(wx[j], s[j], v);
    }
    const size_t cellq = (size_t)cell * w0 + q;
    blk[KIND == 1 ? ((size_t)hd * n + a) * cells * w0 + cellq : ((size_t)hd * cells * w0 + cellq) * n + a] = live * v;
  }
}

// ---------------------------------------------------------------------------
// DWC parameter gradients: dw[c][tap] = sum over batch and tokens of dO[y,x,c] V[y + p, x + q, c], db[c] = sum dO.
// A thread owns a 16-byte piece of the channels of an image column and walks down its rows with the 3 x 3 neighbourhood of V in
// registers, so that a row costs three 16-byte reads of V (two of them shared with the neighbouring columns through
// L1) and one of dO; CHP = 16-byte pieces per token rounded up to a power of two.  The lanes of a block are added by
// a fixed tree, the blocks by dwc_param_sum_kernel.
// grid = (slices, heads); slice = 256 / CHP (column, row segment, image) items.
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

template <class E, int CHP>
__global__ __launch_bounds__(256) void dwc_param_kernel(const typename Piece<E>::S* __restrict__ V,
                                                        const typename Piece<E>::S* __restrict__ dO,
                                                        float* __restrict__ part, int heads, int d, Layout lay, int gh, int gw,
                                                        int segs, int seg_len, int items) {
  using S = typename Piece<E>::S;
  constexpr int P = Piece<E>::kCount;
  __shared__ float red[4][CHP][10 * P];
  const int hd = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int ch = tid % CHP;
  const int item = blockIdx.x * (256 / CHP) + tid / CHP;
  float acc[10][P];
#pragma unroll
  for (int k = 0; k < 10; ++k)
#pragma unroll
    for (int i = 0; i < P; ++i) acc[k][i] = 0.0f;
  if (item < items && ch * P < d) {
    const int x = item % gw, s = item / gw % segs, b = item / gw / segs;
    const int u = b * heads + hd, pitch = lay.pitch(gw);
    const S* v = V + lay.in_unit(u, heads) + ch * P;
    const S* g = dO + lay.out_unit(u, heads) + ch * P;
    const int y0 = s * seg_len, y1 = min(gh, y0 + seg_len);
    float win[3][3][P];      // rows y - 1, y, y + 1 (rotating), columns x - 1 .. x + 1
    auto load_row = [&](int y, float (&o)[3][P]) {
      u32x4 p[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const int xx = x + q - 1;
        p[q] = u32x4{0u, 0u, 0u, 0u};
        if (y >= 0 && y < gh && xx >= 0 && xx < gw) p[q] = *reinterpret_cast<const u32x4*>(v + ((size_t)y * pitch + xx) * lay.sn);
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) Piece<E>::unpack(p[q], o[q]);
    };
    auto row = [&](int y, const float (&a)[3][P], const float (&m)[3][P], float (&z)[3][P]) {
      const u32x4 gp = *reinterpret_cast<const u32x4*>(g + ((size_t)y * pitch + x) * lay.on);
      load_row(y + 1, z);
      float gv[P];
      Piece<E>::unpack(gp, gv);
#pragma unroll
      for (int i = 0; i < P; ++i) acc[9][i] += gv[i];
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < P; ++i) {
          acc[q][i] = fmaf(gv[i], a[q][i], acc[q][i]);
          acc[3 + q][i] = fmaf(gv[i], m[q][i], acc[3 + q][i]);
          acc[6 + q][i] = fmaf(gv[i], z[q][i], acc[6 + q][i]);
        }
    };
    load_row(y0 - 1, win[0]);
    load_row(y0, win[1]);
    int y = y0;
    for (; y + 3 <= y1; y += 3) {
      row(y, win[0], win[1], win[2]);
      row(y + 1, win[1], win[2], win[0]);
      row(y + 2, win[2], win[0], win[1]);
    }
    if (y < y1) row(y, win[0], win[1], win[2]);
    if (y + 1 < y1) row(y + 1, win[1], win[2], win[0]);
  }
#pragma unroll
  for (int k = 0; k < 10; ++k)
#pragma unroll
    for (int i = 0; i < P; ++i) {
      float t = acc[k][i];
#pragma unroll
      for (int o = CHP; o < 64; o <<= 1) t += __shfl_xor(t, o, 64);
      acc[k][i] = t;
    }
  if (lane < CHP)
#pragma unroll
    for (int k = 0; k < 10; ++k)
#pragma unroll
      for (int i = 0; i < P; ++i) red[w][lane][i * 10 + k] = acc[k][i];
  __syncthreads();
  for (int i = tid; i < d * 10; i += 256)      // channel-major, ten sums each
    part[((size_t)hd * gridDim.x + blockIdx.x) * d * 10 + i] =
        (red[0][i / (10 * P)][i % (10 * P)] + red[1][i / (10 * P)][i % (10 * P)]) + (red[2][i / (10 * P)][i % (10 * P)] + red[3][i / (10 * P)][i % (10 * P)]);
}

// one wave per (head, channel): lane l adds the slices l, l + 64, ... in order, the lanes are added by a fixed tree
__global__ __launch_bounds__(64) void dwc_param_total_kernel(const float* __restrict__ part, float* __restrict__ dw,
                                                             float* __restrict__ db, int d, int slices) {
  const int c = blockIdx.x, hd = blockIdx.y, lane = threadIdx.x;
  float acc[10];
#pragma unroll
  for (int k = 0; k < 10; ++k) acc[k] = 0.0f;
  for (int s = lane; s < slices; s += 64) {
    const float* q = part + (((size_t)hd * slices + s) * d + c) * 10;
#pragma unroll
    for (int k = 0; k < 10; ++k) acc[k] += q[k];
  }
#pragma unroll
  for (int k = 0; k < 10; ++k) acc[k] = wave_sum(acc[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 9; ++k) dw[((size_t)hd * d + c) * 9 + k] = acc[k];
    if (db) db[(size_t)hd * d + c] = acc[9];
  }
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

hipError_t launch_backward_bias_tables(const Problem& p, int kind, int cells, int ld, float* ta, float* tx, float* rows,
                                       YInfo* yi, hipStream_t st) {
  const int wp = (p.gw + 15) / 16 * 16;
  const size_t tcount = (size_t)p.heads * cells * (wp / 4) * (ld / 4), rcount = rows ? (size_t)p.heads * p.gh * (ld / 4) : 0;
  const unsigned tb = (unsigned)((tcount + 255) / 256), rb = (unsigned)((rcount + 255) / 256), yb = (unsigned)((p.gh + 255) / 256);
  const dim3 grid(tb + rb + yb);
  if (kind == 1)
    bias_tables_kernel<1><<<grid, dim3(256), 0, st>>>(p.b1, ta, tx, rows, yi, p.heads, p.n, p.gh, p.gw, cells, ld, tb, rb);
  else
    bias_tables_kernel<2><<<grid, dim3(256), 0, st>>>(p.b2, ta, tx, rows, yi, p.heads, p.n, p.gh, p.gw, cells, ld, tb, rb);
  return hipGetLastError();
}

hipError_t launch_backward_bias_grads(const Problem& p, int kind, const BiasGradParts& q, int h0, int w0, float* col,
                                      float* row, float* blk, hipStream_t st) {
  const int batch = p.units / p.heads, wp = (p.gw + 15) / 16 * 16;
  const size_t per_cell = (size_t)(wp / 4) * q.ld;
  const float* sum = q.gt;      // one unit per head and one segment: the parts are the sums
  if ((col || blk) && (batch > 1 || q.segs > 1)) {
    const size_t count = (size_t)p.heads * q.cells * per_cell;
    bias_grad_sum_kernel<<<dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st>>>(
        reinterpret_cast<const f32x4*>(q.gt), reinterpret_cast<f32x4*>(q.sum), batch, p.heads, q.segs, q.seg_len, p.gh, q.cells,
        per_cell);
    sum = q.sum;
  }
  const unsigned cb = col ? (unsigned)(((size_t)p.heads * p.gw * p.n + 255) / 256) : 0;
  const unsigned rb = row ? (unsigned)(((size_t)p.heads * p.gh * p.n + 255) / 256) : 0;
  const unsigned bb = blk ? (unsigned)(((size_t)p.heads * h0 * w0 * p.n + 255) / 256) : 0;
  if (cb + rb + bb == 0) return hipGetLastError();
  const float live = (kind == 1 ? p.N : p.n) > 1 ? 1.0f : 0.0f;
  if (kind == 1)
    bias_grad_out_kernel<1><<<dim3(cb + rb + bb), dim3(256), 0, st>>>(reinterpret_cast<const f32x4*>(sum), q.gr, col, row, blk,
                                                                     batch, p.heads, p.n, p.gh, p.gw, q.cells, w0, q.ld, live, cb,
                                                                     rb);
  else
    bias_grad_out_kernel<2><<<dim3(cb + rb + bb), dim3(256), 0, st>>>(reinterpret_cast<const f32x4*>(sum), q.gr, col, row, blk,
                                                                     batch, p.heads, p.n, p.gh, p.gw, q.cells, w0, q.ld, live, cb,
                                                                     rb);
  return hipGetLastError();
}

size_t dwc_param_part_floats(const Problem& p) { return (size_t)p.heads * dwc_plan(p).slices * p.d * 10; }

hipError_t launch_dwc_param_grads(const Problem& p, const void* V, const void* dO, float* part, float* dw, float* db,
                                  hipStream_t st) {
  const DwcPlan q = dwc_plan(p);
  const dim3 grid(q.slices, p.heads);
  auto go = [&](auto kernel, auto elem) {
    using S = typename Piece<decltype(elem)>::S;
    kernel<<<grid, dim3(256), 0, st>>>((const S*)V, (const S*)dO, part, p.heads, p.d, p.lay, p.gh, p.gw, q.segs, q.seg_len,
                                       q.items);
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
  dwc_param_total_kernel<<<dim3(p.d, p.heads), dim3(64), 0, st>>>(part, dw, db, p.d, q.slices);
  return hipGetLastError();
}

}  // namespace aa
