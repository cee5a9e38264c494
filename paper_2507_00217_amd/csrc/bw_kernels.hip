// Bandwidth-bound kernels of the stage: LayerNorm / RMSNorm forward and backward
// (wavefront reductions, rows held in registers so HBM is read once), GELU /
// SwiGLU forward and backward, fill and copy.  All accesses are 16-byte vectors.
// Norm-parameter gradients are produced here, at B time, through per-workgroup
// partial sums reduced in a fixed order (no atomics), so results do not depend
// on scheduling.
#include "common.h"

#include <mutex>

namespace stg {

template <typename T> struct Vec {
  static constexpr int N = 16 / sizeof(T);
  union { uint4 raw; T v[16 / sizeof(T)]; };
};

template <typename T> __device__ __forceinline__ Vec<T> ldv(const T* p) {
  Vec<T> r; r.raw = *reinterpret_cast<const uint4*>(p); return r;
}
template <typename T> __device__ __forceinline__ void stv(T* p, const Vec<T>& r) {
  *reinterpret_cast<uint4*>(p) = r.raw;
}

// V consecutive elements starting at element offset `off` of a row that is stored either in T or (wide) in fp32
template <typename T>
__device__ __forceinline__ void ld_row(float (&dst)[Vec<T>::N], const void* base, int64_t off, bool wide) {
  constexpr int V = Vec<T>::N;
  if (wide && sizeof(T) != 4) {
    const float4* p = reinterpret_cast<const float4*>((const float*)base + off);
#pragma unroll
    for (int q = 0; q < V / 4; ++q) { float4 t = p[q]; dst[4 * q] = t.x; dst[4 * q + 1] = t.y; dst[4 * q + 2] = t.z; dst[4 * q + 3] = t.w; }
  } else {
    Vec<T> t = ldv((const T*)base + off);
#pragma unroll
    for (int e = 0; e < V; ++e) dst[e] = to_f32(t.v[e]);
  }
}
template <typename T>
__device__ __forceinline__ void st_row(void* base, int64_t off, const float (&src)[Vec<T>::N], bool wide) {
  constexpr int V = Vec<T>::N;
  if (wide && sizeof(T) != 4) {
    float4* p = reinterpret_cast<float4*>((float*)base + off);
#pragma unroll
    for (int q = 0; q < V / 4; ++q) p[q] = make_float4(src[4 * q], src[4 * q + 1], src[4 * q + 2], src[4 * q + 3]);
  } else {
    Vec<T> o;
#pragma unroll
    for (int e = 0; e < V; ++e) o.v[e] = from_f32<T>(src[e]);
    stv((T*)base + off, o);
  }
}

constexpr int NORM_THREADS = 256;
constexpr int NORM_MAXCH = 4;          // 16-byte chunks per thread: d <= 256*4*(16/sizeof(T))
constexpr int NORM_PARTIAL_ROWS = 512;   // backward: partial rows the caller's scratch holds, at most this many workgroups
int norm_partial_rows() { return NORM_PARTIAL_ROWS; }

__device__ __forceinline__ float wg_sum(float v, float* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// out = (x - mean) * rstd * gamma + beta   |   out = x * rstd * gamma; x_wide, if given, receives x in fp32 on the way
template <typename T, int KIND>
__global__ __launch_bounds__(NORM_THREADS) void norm_fwd_kernel(NormArgs n) {
  constexpr int V = Vec<T>::N;
  __shared__ float red[4];
  const int row = blockIdx.x;
  const int64_t roff = (int64_t)row * n.d;
  T* out = (T*)n.out + roff;
  const int nvec = n.d / V;
  float xv[NORM_MAXCH][V];
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < NORM_MAXCH; ++c) {
    const int vi = threadIdx.x + c * NORM_THREADS;
    if (vi < nvec) {
      ld_row<T>(xv[c], n.x, roff + vi * V, n.x_f32);
      if (n.x_wide) st_row<T>(n.x_wide, roff + vi * V, xv[c], true);
#pragma unroll
      for (int e = 0; e < V; ++e) s += (KIND == 0) ? xv[c][e] : xv[c][e] * xv[c][e];
    }
  }
  float mean = 0.f, rstd;
  const float inv_d = 1.f / (float)n.d;
  if (KIND == 0) {
    mean = wg_sum(s, red) * inv_d;
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < NORM_MAXCH; ++c)
      if (threadIdx.x + c * NORM_THREADS < nvec)
#pragma unroll
        for (int e = 0; e < V; ++e) { float t = xv[c][e] - mean; q += t * t; }
    rstd = rsqrtf(wg_sum(q, red) * inv_d + n.eps);
  } else {
    rstd = rsqrtf(wg_sum(s, red) * inv_d + n.eps);
  }
  if (threadIdx.x == 0) { n.stats[2 * row] = mean; n.stats[2 * row + 1] = rstd; }
#pragma unroll
  for (int c = 0; c < NORM_MAXCH; ++c) {
    const int vi = threadIdx.x + c * NORM_THREADS;
    if (vi < nvec) {
      Vec<T> g = ldv((const T*)n.gamma + vi * V), b, o;
      if (KIND == 0) b = ldv((const T*)n.beta + vi * V);
#pragma unroll
      for (int e = 0; e < V; ++e) {
        float y = (xv[c][e] - mean) * rstd * to_f32(g.v[e]);
        if (KIND == 0) y += to_f32(b.v[e]);
        o.v[e] = from_f32<T>(y);
      }
      stv(out + vi * V, o);
    }
  }
}

// dx = resid + rstd * (dxhat - mean(dxhat) - xhat * mean(dxhat * xhat)),  dxhat = dout * gamma
// (the mean(dxhat) term is absent for RMSNorm); per-workgroup partial sums of
// dgamma = sum_rows dout * xhat and dbeta = sum_rows dout go to n.partial.
//
// Bound by HBM, 8 bytes per element (16 with an fp32 residual stream), as long as enough rows are in flight.  A row takes up to
// four wavefronts, piece c of thread t being 16-byte piece t + 256 c of the row, and CH <= 4 pieces per thread (fewer wavefronts
// for rows of less than 256 pieces): the row sums are then the same whatever else the workgroup does.  Rows of one piece per
// thread stand side by side in workgroups of up to eight wavefronts.  Both row sums cross the workgroup in one exchange, xhat and
// dxhat are formed again from the raw row rather than kept, and where registers allow (PF) the next row's loads are issued before
// this one is reduced.  With its column sums and operands from HBM, against one row of 256 threads at a time and two exchanges:
// LayerNorm 4096 x 5120 in bf16 72 -> 45.6 us, 2048 x 2048 with an fp32 residual stream 24 -> 17.5; RMSNorm 2048 x 6144 in bf16 34.6 ->
// 27.4, 4096 x 4096 with an fp32 residual stream, at 4.8 TB/s already, 55 -> 56.
template <typename T, bool WIDE> struct RowPiece { static constexpr int W = WIDE ? Vec<T>::N / 4 : 1; uint4 v[W]; };
template <typename T, bool WIDE>
__device__ __forceinline__ RowPiece<T, WIDE> ld_piece(const void* base, int64_t off) {
  RowPiece<T, WIDE> r;
  const uint4* p = reinterpret_cast<const uint4*>((const char*)base + off * (WIDE ? 4 : sizeof(T)));
#pragma unroll
  for (int q = 0; q < RowPiece<T, WIDE>::W; ++q) r.v[q] = p[q];
  return r;
}
template <typename T, bool WIDE> __device__ __forceinline__ float at_piece(const RowPiece<T, WIDE>& r, int e) {
  if constexpr (WIDE || sizeof(T) == 4) {
    const uint4 q = r.v[WIDE ? e / 4 : 0];
    return __uint_as_float((e & 3) == 0 ? q.x : (e & 3) == 1 ? q.y : (e & 3) == 2 ? q.z : q.w);
  } else {
    Vec<T> t; t.raw = r.v[0];
    return to_f32(t.v[e]);
  }
}

constexpr int NB_THREADS = 512;
// XW / RW: x / resid is stored in fp32 although T is not
template <typename T, int KIND, bool XW, bool RW, int CH, bool PF, bool SIDE>
__global__ __launch_bounds__(SIDE ? NB_THREADS : NORM_THREADS) void norm_bwd_kernel(NormArgs n, int tpr) {
  constexpr int V = Vec<T>::N;
  extern __shared__ float col_sums[];                    // [row groups - 1][2][d]: the first group's stay in its registers
  __shared__ float red[2][NB_THREADS / 64][2];
  const int nvec = n.d / V, ngrp = blockDim.x / tpr, wpr = tpr >> 6;
  const int grp = threadIdx.x / tpr, t = threadIdx.x % tpr, wave = threadIdx.x >> 6;
  float dg[CH][V], db[CH][V];
  Vec<T> gam[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int vi = t + c * tpr;
    gam[c] = ldv((const T*)n.gamma + (vi < nvec ? vi : 0) * V);
#pragma unroll
    for (int e = 0; e < V; ++e) dg[c][e] = db[c][e] = 0.f;
  }
  const float inv_d = 1.f / (float)n.d;
  RowPiece<T, XW> x[CH], xn[CH];
  RowPiece<T, RW> rs[CH], rsn[CH];
  Vec<T> dv[CH], dvn[CH];
  float mean = 0.f, rstd = 0.f, mean_n = 0.f, rstd_n = 0.f;
  // rows past the end are read as the last one and leave no trace
  auto load = [&](int row) __attribute__((always_inline)) {
    const int r = min(row, n.rows - 1);
    const int64_t roff = (int64_t)r * n.d;
    mean_n = n.stats[2 * r]; rstd_n = n.stats[2 * r + 1];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int vi = t + c * tpr;
      const int64_t off = roff + (vi < nvec ? vi : 0) * V;
      xn[c] = ld_piece<T, XW>(n.x, off);
      dvn[c] = ldv((const T*)n.dout + off);
      if (n.resid) rsn[c] = ld_piece<T, RW>(n.resid, off);
    }
  };
  const int step = gridDim.x * ngrp;
  int row0 = blockIdx.x * ngrp;
  if (PF) load(row0 + grp);
  for (int it = 0; row0 < n.rows; row0 += step, ++it) {
    const int row = row0 + grp;
    if (!PF) load(row);
    mean = mean_n; rstd = rstd_n;
#pragma unroll
    for (int c = 0; c < CH; ++c) { x[c] = xn[c]; dv[c] = dvn[c]; rs[c] = rsn[c]; }
    if (PF && row0 + step < n.rows) load(row + step);
    const bool live = row < n.rows;
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (live && t + c * tpr < nvec) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const float xhat = (at_piece<T, XW>(x[c], e) - mean) * rstd, d = to_f32(dv[c].v[e]), dx = d * to_f32(gam[c].v[e]);
          dg[c][e] += d * xhat;
          if (KIND == 0) { db[c][e] += d; s1 += dx; }
          s2 += dx * xhat;
        }
      }
    for (int o = 32; o > 0; o >>= 1) {
      if (KIND == 0) s1 += __shfl_xor(s1, o, 64);
      s2 += __shfl_xor(s2, o, 64);
    }
    if (wpr > 1) {                                       // two sets of slots in turn: one barrier per row
      if ((threadIdx.x & 63) == 0) { red[it & 1][wave][0] = s1; red[it & 1][wave][1] = s2; }
      __syncthreads();
      s1 = s2 = 0.f;
      for (int k = 0; k < wpr; ++k) { s1 += red[it & 1][grp * wpr + k][0]; s2 += red[it & 1][grp * wpr + k][1]; }
    }
    float m1, m2;
    {
#pragma clang fp contract(off)                           // rounded before they are subtracted
      m1 = s1 * inv_d; m2 = s2 * inv_d;
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int vi = t + c * tpr;
      if (live && vi < nvec) {
        const int64_t off = (int64_t)row * n.d + vi * V;
        float o[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const float xhat = (at_piece<T, XW>(x[c], e) - mean) * rstd;
          float dxhat;
          {
#pragma clang fp contract(off)                           // the rounded product, as in the sums
            dxhat = to_f32(dv[c].v[e]) * to_f32(gam[c].v[e]);
          }
          o[e] = (dxhat - m1 - xhat * m2) * rstd;
          if (n.resid) o[e] += at_piece<T, RW>(rs[c], e);
        }
        st_row<T>(n.out, off, o, n.out_f32);
        if (n.out_lp) st_row<T>(n.out_lp, off, o, false);
        if (!RW && n.resid_copy) *reinterpret_cast<uint4*>((T*)n.resid_copy + off) = rs[c].v[0];
      }
    }
  }
  if (SIDE && ngrp > 1) {                                // the row groups' column sums, in order
    float* cs = col_sums + (int64_t)(grp - 1) * 2 * n.d;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int vi = t + c * tpr;
      if (grp > 0 && vi < nvec)
#pragma unroll
        for (int e = 0; e < V; ++e) { cs[vi * V + e] = dg[c][e]; if (KIND == 0) cs[n.d + vi * V + e] = db[c][e]; }
    }
    __syncthreads();
    if (grp != 0) return;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int vi = t + c * tpr;
      if (vi < nvec)
        for (int g = 1; g < ngrp; ++g)
#pragma unroll
          for (int e = 0; e < V; ++e) {
            dg[c][e] += col_sums[(int64_t)(g - 1) * 2 * n.d + vi * V + e];
            if (KIND == 0) db[c][e] += col_sums[(int64_t)(g - 1) * 2 * n.d + n.d + vi * V + e];
          }
    }
  }
  float* pg = n.partial + (int64_t)blockIdx.x * 2 * n.d;
  float* pb = pg + n.d;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int vi = t + c * tpr;
    if (vi < nvec)
#pragma unroll
      for (int q = 0; q < V / 4; ++q) {
        *reinterpret_cast<float4*>(pg + vi * V + 4 * q) = make_float4(dg[c][4 * q], dg[c][4 * q + 1], dg[c][4 * q + 2], dg[c][4 * q + 3]);
        if (KIND == 0) *reinterpret_cast<float4*>(pb + vi * V + 4 * q) = make_float4(db[c][4 * q], db[c][4 * q + 1], db[c][4 * q + 2], db[c][4 * q + 3]);
      }
  }
}

// dst[col] += sum over a job's rows, in a fixed order, for all jobs of the list (norm-parameter and bias gradients of a layer) in
// one launch: 64 columns per workgroup, the rows dealt out to SUM_WAVES wavefronts, whose shares wavefront 0 adds in order.
// What bounds it is a few microseconds of memory latency, not bandwidth, so every job has its loads in flight together: partial
// sums take one row per wavefront and load (coalesced 256 bytes), 16 of them at once; gradient rows (below) 16 bytes per lane,
// 8 (bf16) or 4 rows per wavefront and load, 8 at once, that is up to 1024 or 512 rows without a second wait.
constexpr int SUM_WAVES = 16;
template <typename T>
__device__ __forceinline__ void gradient_row_sums(const ColSum& j, int col0, int w, int lane, float* share) {
  constexpr int V = Vec<T>::N, C = 64 / V, R = 64 / C, U = 8;   // C lanes across the 64 columns, R rows at once
  const int col = col0 + (lane % C) * V;
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.f;
  if (col < j.cols)                                            // cols is a multiple of V
    for (int r0 = w * R + lane / C; r0 < j.parts; r0 += SUM_WAVES * R * U) {
      Vec<T> v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * SUM_WAVES * R;
        if (r < j.parts) v[u] = ldv((const T*)j.part + (int64_t)r * j.stride + col);
        else v[u] = Vec<T>{};
      }
#pragma unroll
      for (int e = 0; e < V; ++e)
        acc[e] += ((to_f32(v[0].v[e]) + to_f32(v[1].v[e])) + (to_f32(v[2].v[e]) + to_f32(v[3].v[e]))) +
                  ((to_f32(v[4].v[e]) + to_f32(v[5].v[e])) + (to_f32(v[6].v[e]) + to_f32(v[7].v[e])));
    }
#pragma unroll
  for (int e = 0; e < V; ++e) {
#pragma unroll
    for (int o = C; o < 64; o <<= 1) acc[e] += __shfl_xor(acc[e], o);
    if (lane < C) share[lane * V + e] = acc[e];
  }
}

// (Two workgroups to a CU: 64 registers.  With 67 more than 256 workgroups took two rounds: a bias gradient of 2048 x 18432 in two
// steps 17.9 instead of 17.2 us.)
__global__ __launch_bounds__(SUM_WAVES * 64, 8) void col_sum_kernel(ColSumList l) {
  __shared__ float sums[SUM_WAVES][64];
  int ji = 0;
  while (ji + 1 < l.n && (int)blockIdx.x >= l.first[ji + 1]) ++ji;
  const ColSum j = l.j[ji];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col0 = ((int)blockIdx.x - l.first[ji]) * 64, col = col0 + lane;
  if (j.rows_of == COL_SUM_BF16_ROWS) gradient_row_sums<bf16>(j, col0, w, lane, sums[w]);
  else if (j.rows_of == COL_SUM_F32_ROWS) gradient_row_sums<float>(j, col0, w, lane, sums[w]);
  else {
    float s = 0.f;
    if (col < j.cols) {
      constexpr int U = 16;
      const float* part = (const float*)j.part;
      for (int p0 = w; p0 < j.parts; p0 += SUM_WAVES * U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int p = p0 + u * SUM_WAVES;
          v[u] = p < j.parts ? part[(int64_t)p * j.stride + col] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) s += v[u];
      }
    }
    sums[w][lane] = s;
  }
  __syncthreads();
  if (w == 0 && col < j.cols) {
    float r = sums[0][lane];
#pragma unroll
    for (int k = 1; k < SUM_WAVES; ++k) r += sums[k][lane];
    j.dst[col] += r;
  }
}

hipError_t col_sums_add(ColSumList& l, hipStream_t s) {
  if (l.n == 0) return hipSuccess;
  int total = 0;
  for (int i = 0; i < l.n; ++i) { l.first[i] = total; total += (l.j[i].cols + 63) / 64; }
  hipLaunchKernelGGL(col_sum_kernel, dim3(total), dim3(SUM_WAVES * 64), 0, s, l);
  return hipGetLastError();
}

template <typename T>
static bool norm_shape_ok(const NormArgs& n) {
  constexpr int V = 16 / sizeof(T);
  return n.d % V == 0 && n.d / V <= NORM_THREADS * NORM_MAXCH && n.rows > 0;
}

template <typename T>
static hipError_t norm_fwd_t(const NormArgs& n, hipStream_t s) {
  if (!norm_shape_ok<T>(n)) return hipErrorInvalidValue;
  if (n.kind == 0) hipLaunchKernelGGL((norm_fwd_kernel<T, 0>), dim3(n.rows), dim3(NORM_THREADS), 0, s, n);
  else hipLaunchKernelGGL((norm_fwd_kernel<T, 1>), dim3(n.rows), dim3(NORM_THREADS), 0, s, n);
  return hipGetLastError();
}

// Rows side by side (SIDE): with one piece per thread, and in fp32, whose pieces are half as many elements, as many rows as eight
// wavefronts hold, one such workgroup per CU -- half the partial rows of two workgroups of half the size (us, two against
// one; 2048 x 2048 with an fp32 residual stream: 18.6 / 17.8; 4096 x 2048 in bf16: 20.2 / 19.1; 448 x 4096 in fp32: 14.1 / 12.7).
// Other rows go one to a workgroup, two workgroups per CU (4096 x 4096 in bf16: 35.2, two rows in one workgroup per CU 38.8).
// Prefetch (PF): in fp32 and with one or two pieces (4096 x 3072 in bf16 30.5, without 34.4; 4096 x 4096 with an fp32 residual stream
// between its neighbours in a layer 34.2 / 38.3); beyond that its registers cost more rows in flight than it hides (4096 x 5120 with
// an fp32 residual stream: 74.8 / 72.4; 2048 x 6144: 52.2 / 50.4; 4096 x 8192 would spill).
template <typename T, int KIND, bool XW, bool RW, int CH>
static hipError_t norm_bwd_launch(const NormArgs& n, hipStream_t s, int* parts) {
  constexpr bool SIDE = CH == 1 || sizeof(T) == 4, PF = SIDE || CH == 2;
  const int units = (n.d / Vec<T>::N + 63) / 64, tpr = 64 * (units < 4 ? units : 4);
  int ngrp = SIDE ? NB_THREADS / tpr : 1;
  const int n_cu = cu_count();
  if (ngrp > 1 && n.rows < n_cu * ngrp) ngrp = NORM_THREADS / tpr;
  const int fill = SIDE ? n_cu : 2 * n_cu, cap = fill < NORM_PARTIAL_ROWS ? fill : NORM_PARTIAL_ROWS, want = (n.rows + ngrp - 1) / ngrp;
  *parts = want < cap ? want : cap;
  const size_t lds = (size_t)(ngrp - 1) * 2 * n.d * sizeof(float);       // at most 32 KiB: ngrp * d <= CH * V * NB_THREADS
  hipLaunchKernelGGL((norm_bwd_kernel<T, KIND, XW, RW, CH, PF, SIDE>), dim3(*parts), dim3(ngrp * tpr), lds, s, n, tpr);
  return hipGetLastError();
}
template <typename T, int KIND, bool XW, bool RW>
static hipError_t norm_bwd_width(const NormArgs& n, hipStream_t s, int* parts) {
  switch ((n.d / Vec<T>::N + NORM_THREADS - 1) / NORM_THREADS) {                 // pieces per thread
    case 1: return norm_bwd_launch<T, KIND, XW, RW, 1>(n, s, parts);
    case 2: return norm_bwd_launch<T, KIND, XW, RW, 2>(n, s, parts);
    case 3: return norm_bwd_launch<T, KIND, XW, RW, 3>(n, s, parts);
    default: return norm_bwd_launch<T, KIND, XW, RW, 4>(n, s, parts);
  }
}
template <typename T, int KIND>
static hipError_t norm_bwd_pick(const NormArgs& n, hipStream_t s, int* parts) {
  if constexpr (sizeof(T) == 2) {
    if (n.x_f32 && n.resid_f32 && n.resid) return norm_bwd_width<T, KIND, true, true>(n, s, parts);
    if (n.x_f32) return norm_bwd_width<T, KIND, true, false>(n, s, parts);
    if (n.resid_f32 && n.resid) return hipErrorInvalidValue;       // no caller: the residual stream is fp32 where x is
  }
  return norm_bwd_width<T, KIND, false, false>(n, s, parts);
}
template <typename T>
static hipError_t norm_bwd_t(const NormArgs& n, hipStream_t s, int* parts) {
  if (!norm_shape_ok<T>(n)) return hipErrorInvalidValue;
  return n.kind == 0 ? norm_bwd_pick<T, 0>(n, s, parts) : norm_bwd_pick<T, 1>(n, s, parts);
}

hipError_t norm_fwd(DType dt, const NormArgs& n, hipStream_t s) {
  return dt == DT_F32 ? norm_fwd_t<float>(n, s) : norm_fwd_t<bf16>(n, s);
}
hipError_t norm_bwd_rows(DType dt, const NormArgs& n, hipStream_t s, int* parts) {
  return dt == DT_F32 ? norm_bwd_t<float>(n, s, parts) : norm_bwd_t<bf16>(n, s, parts);
}
void norm_col_sums(const NormArgs& n, int parts, ColSumList* l) {
  l->j[l->n++] = ColSum{n.partial, (int64_t)2 * n.d, n.d, parts, n.dgamma, COL_SUM_PARTS};
  if (n.kind == 0) l->j[l->n++] = ColSum{n.partial + n.d, (int64_t)2 * n.d, n.d, parts, n.dbeta, COL_SUM_PARTS};
}
hipError_t norm_bwd(DType dt, const NormArgs& n, hipStream_t s) {
  int parts = 0;
  const hipError_t e = norm_bwd_rows(dt, n, s, &parts);
  if (e != hipSuccess) return e;
  ColSumList l{};
  norm_col_sums(n, parts, &l);
  return col_sums_add(l, s);
}

// Norm backward for callers that cannot allocate device memory: the per-workgroup partial sums of dgamma / dbeta go to
// a fixed array in the library's own device image instead of a caller-provided buffer.  Every GPU the library runs on
// holds its own copy of the array, at its own address, until the process ends; `scratch` in host code is only a handle
// to the symbol, so the device address is looked up once per device and that pointer is what the kernels are given.
// The kernels write every partial they later read, so nothing has to be cleared between calls; two calls that
// overlap on one GPU (different streams) would race on the array.
constexpr int NOALLOC_MAX_D = 8192;
constexpr int NOALLOC_MAX_DEVICES = 64;
static __device__ __align__(256) float scratch[(size_t)NORM_PARTIAL_ROWS * 2 * NOALLOC_MAX_D];   // 32 MiB

int norm_bwd_noalloc_max_d() { return NOALLOC_MAX_D; }

hipError_t norm_bwd_noalloc(DType dt, const NormArgs& n, hipStream_t s) {
  static std::mutex mu;
  static float* scratch_of[NOALLOC_MAX_DEVICES] = {};
  if (n.d < 1 || n.d > NOALLOC_MAX_D) return hipErrorInvalidValue;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
  float* ptr;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!scratch_of[dev]) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));     // the current device's copy
      if (e != hipSuccess) return e;
      if (!p) return hipErrorInvalidSymbol;
      scratch_of[dev] = (float*)p;
    }
    ptr = scratch_of[dev];
  }
  NormArgs m = n;
  m.partial = ptr;
  return norm_bwd(dt, m, s);
}

// ---------------------------------------------------------------------------
// Gradient of a linear map's bias: the column sums of its dZ, added to the fp32 accumulator, with a fixed summation order (no
// atomics).  Up to a number of rows (bias_grad_direct) col_sum_kernel sums dZ itself, in the launch that also adds the norms' partial sums.
// Beyond that two steps: BIAS_PARTS row ranges are summed by one workgroup each per 32 x (16 / sizeof(T)) columns -- 8 row
// lanes per column group, combined through LDS in lane order -- then col_sum_kernel adds the parts.  The four maps of a
// layer go out together.
// The line: a workgroup of the one step owns its 64 columns alone, so its time grows with the rows, where the two steps spread
// them over 64 workgroups but pay a second launch (us, one step / two).
//   rows that start on 128-byte lines, up to 16384 columns: 2048 rows (bf16, 5120 columns, 1024 rows 4.4 / 6.4, 2048 5.5 / 7.2; 12288
//     columns, 2048 rows 10.5 / 12.5; fp32, 5120 columns, 2048 rows 9.8 / 11.1; 1920 columns, 1800 rows 5.8 / 6.2, 2048 6.2 / 6.3, 3072 9.4 / 7.4)
//   wider: 1024, there are workgroups enough to be past the latency (18432 columns, bf16, 1024 rows 11.5 / 12.0, 2048 18.0 / 17.1; fp32, 2048
//     rows 27.7 / 26.3)
//   off the lines: 1024, and 512 of more than 8192 columns; the 128 bytes of a workgroup's columns are then two lines, each fetched twice
//     (bf16, 5144 columns, 1024 rows 5.4 / 6.4, 2048 8.7 / 7.6; 12280 columns, 1024 rows 9.7 / 9.2; fp32, 3576 columns, 1024 rows 4.7 / 6.8, 1800 9.3 /
//     7.5)
// ---------------------------------------------------------------------------
constexpr int BIAS_PARTS = 64;
size_t bias_grad_partial_bytes(int n) { return n > 0 ? (size_t)BIAS_PARTS * n * sizeof(float) : 0; }

template <typename T>
__global__ __launch_bounds__(256) void bias_grad_partial_kernel(BiasGradList l) {
  constexpr int V = Vec<T>::N;
  __shared__ float red[8][32 * V];
  int ji = 0;
  while (ji + 1 < l.n && (int)blockIdx.x >= l.first[ji + 1]) ++ji;
  const BiasGrad j = l.j[ji];
  const T* dz = (const T*)j.dz;
  const int cg = threadIdx.x & 31, rl = threadIdx.x >> 5;
  const int col = (((int)blockIdx.x - l.first[ji]) * 32 + cg) * V;
  const int per = (l.rows + BIAS_PARTS - 1) / BIAS_PARTS;
  const int r0 = blockIdx.y * per, r1 = min(l.rows, r0 + per);
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.f;
  if (col < j.cols)
    for (int r = r0 + rl; r < r1; r += 8) {
      Vec<T> v = ldv(dz + (int64_t)r * j.ld + col);
#pragma unroll
      for (int e = 0; e < V; ++e) acc[e] += to_f32(v.v[e]);
    }
#pragma unroll
  for (int e = 0; e < V; ++e) red[rl][cg * V + e] = acc[e];
  __syncthreads();
  if (rl == 0 && col < j.cols) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
      float s = red[0][cg * V + e];
#pragma unroll
      for (int k = 1; k < 8; ++k) s += red[k][cg * V + e];
      j.part[(int64_t)blockIdx.y * j.cols + col + e] = s;
    }
  }
}

bool bias_grad_direct(DType dt, const BiasGradList& l) {
  const int64_t es = dt == DT_F32 ? 4 : 2;
  bool lines = true;
  int64_t cols = 0;
  for (int i = 0; i < l.n; ++i) {
    lines = lines && ((uintptr_t)l.j[i].dz & 127) == 0 && l.j[i].ld * es % 128 == 0;
    cols += l.j[i].cols;
  }
  return l.rows <= (lines ? cols <= 16384 ? 2048 : 1024 : cols <= 8192 ? 1024 : 512);
}
hipError_t bias_grad_rows(DType dt, BiasGradList& l, ColSumList* sums, hipStream_t s) {
  const int V = dt == DT_F32 ? 4 : 8;
  if (l.n == 0) return hipSuccess;
  const bool direct = bias_grad_direct(dt, l);
  int total = 0;
  for (int i = 0; i < l.n; ++i) {
    const BiasGrad& j = l.j[i];
    if (l.rows < 1 || j.cols < 1 || j.cols % V || j.ld % V || !j.dz || !j.part || !j.dbias || ((uintptr_t)j.dz & 15)) return hipErrorInvalidValue;
    l.first[i] = total;
    total += (j.cols / V + 31) / 32;
    if (direct) sums->j[sums->n++] = ColSum{j.dz, j.ld, j.cols, l.rows, j.dbias, dt == DT_BF16 ? COL_SUM_BF16_ROWS : COL_SUM_F32_ROWS};
    else sums->j[sums->n++] = ColSum{j.part, j.cols, j.cols, BIAS_PARTS, j.dbias, COL_SUM_PARTS};
  }
  if (direct) return hipSuccess;
  const dim3 grid(total, BIAS_PARTS);
  if (dt == DT_F32) hipLaunchKernelGGL((bias_grad_partial_kernel<float>), grid, dim3(256), 0, s, l);
  else hipLaunchKernelGGL((bias_grad_partial_kernel<bf16>), grid, dim3(256), 0, s, l);
  return hipGetLastError();
}

hipError_t bias_grad(DType dt, const void* dz, int64_t ld, int rows, int n, float* partial, float* dbias, hipStream_t s) {
  BiasGradList l{};
  l.rows = rows; l.n = 1; l.j[0] = BiasGrad{dz, ld, n, partial, dbias};
  ColSumList sums{};
  const hipError_t e = bias_grad_rows(dt, l, &sums, s);
  return e != hipSuccess ? e : col_sums_add(sums, s);
}

// ---------------------------------------------------------------------------
// activations
// ---------------------------------------------------------------------------
__device__ __forceinline__ float gelu_f(float u) { return 0.5f * u * (1.f + erff(u * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_df(float u) {
  return 0.5f * (1.f + erff(u * 0.70710678118654752f)) + u * 0.39894228040143268f * __expf(-0.5f * u * u);
}
__device__ __forceinline__ float sigmoid_f(float g) { return 1.f / (1.f + __expf(-g)); }

// GELU: a = gelu(z).  SwiGLU: a = silu(z[:, :f]) * z[:, f:]
template <typename T, int KIND>
__global__ __launch_bounds__(256) void act_fwd_kernel(ActArgs a) {
  constexpr int V = Vec<T>::N;
  const int fv = a.f / V;
  const int64_t total = (int64_t)a.rows * fv;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / fv; const int c = (int)(i % fv) * V;
    Vec<T> o;
    if (KIND == 0) {
      Vec<T> u = ldv((const T*)a.z + r * a.f + c);
#pragma unroll
      for (int e = 0; e < V; ++e) o.v[e] = from_f32<T>(gelu_f(to_f32(u.v[e])));
    } else {
      Vec<T> g = ldv((const T*)a.z + r * 2 * a.f + c), u = ldv((const T*)a.z + r * 2 * a.f + a.f + c);
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const float gv = to_f32(g.v[e]);
        o.v[e] = from_f32<T>(gv * sigmoid_f(gv) * to_f32(u.v[e]));
      }
    }
    stv((T*)a.a + r * a.f + c, o);
  }
}

// GELU: z := da * gelu'(z).  SwiGLU: z[:, :f] := da*u*(sg + g*sg*(1-sg)),  z[:, f:] := da*g*sg
template <typename T, int KIND>
__global__ __launch_bounds__(256) void act_bwd_kernel(ActArgs a) {
  constexpr int V = Vec<T>::N;
  const int fv = a.f / V;
  const int64_t total = (int64_t)a.rows * fv;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / fv; const int c = (int)(i % fv) * V;
    Vec<T> da = ldv((const T*)a.da + r * a.f + c);
    if (KIND == 0) {
      T* zp = (T*)a.z + r * a.f + c;
      Vec<T> u = ldv(zp), o;
#pragma unroll
      for (int e = 0; e < V; ++e) o.v[e] = from_f32<T>(to_f32(da.v[e]) * gelu_df(to_f32(u.v[e])));
      stv(zp, o);
    } else {
      T* gp = (T*)a.z + r * 2 * a.f + c; T* up = gp + a.f;
      Vec<T> g = ldv(gp), u = ldv(up), og, ou;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const float gv = to_f32(g.v[e]), uv = to_f32(u.v[e]), d = to_f32(da.v[e]);
        const float sg = sigmoid_f(gv);
        og.v[e] = from_f32<T>(d * uv * (sg + gv * sg * (1.f - sg)));
        ou.v[e] = from_f32<T>(d * gv * sg);
      }
      stv(gp, og); stv(up, ou);
    }
  }
}

template <typename T>
static hipError_t act_t(const ActArgs& a, bool bwd, hipStream_t s) {
  constexpr int V = 16 / sizeof(T);
  if (a.f % V != 0 || a.rows <= 0) return hipErrorInvalidValue;
  const int64_t total = (int64_t)a.rows * (a.f / V);
  const int grid = (int)((total + 255) / 256 < 65536 ? (total + 255) / 256 : 65536);
  if (!bwd) {
    if (a.kind == 0) hipLaunchKernelGGL((act_fwd_kernel<T, 0>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((act_fwd_kernel<T, 1>), dim3(grid), dim3(256), 0, s, a);
  } else {
    if (a.kind == 0) hipLaunchKernelGGL((act_bwd_kernel<T, 0>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((act_bwd_kernel<T, 1>), dim3(grid), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t act_fwd(DType dt, const ActArgs& a, hipStream_t s) {
  return dt == DT_F32 ? act_t<float>(a, false, s) : act_t<bf16>(a, false, s);
}
hipError_t act_bwd(DType dt, const ActArgs& a, hipStream_t s) {
  return dt == DT_F32 ? act_t<float>(a, true, s) : act_t<bf16>(a, true, s);
}

// ---------------------------------------------------------------------------
// fill / copy (kernels rather than memset/memcpy nodes, so that a caller may
// capture a schedule into a HIP graph)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fill_zero_kernel(uint4* p, size_t nvec, float* tail, size_t ntail) {
  const uint4 z = {0, 0, 0, 0};
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (size_t)gridDim.x * 256) p[i] = z;
  if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0.f;
}

hipError_t fill_zero_f32(float* p, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const size_t nvec = n / 4;
  const size_t want = (nvec + 255) / 256;
  const int grid = (int)(want < 1 ? 1 : (want > 16384 ? 16384 : want));
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, s, (uint4*)p, nvec, p + nvec * 4, n - nvec * 4);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void copy_kernel(uint4* dst, const uint4* src, size_t nvec) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

hipError_t copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  if (bytes % 16) return hipErrorInvalidValue;
  const size_t nvec = bytes / 16;
  const size_t want = (nvec + 255) / 256;
  const int grid = (int)(want > 16384 ? 16384 : want);
  hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(256), 0, s, (uint4*)dst, (const uint4*)src, nvec);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Rotary position embedding (the paper's layers are Llama-style): consecutive pairs (2p, 2p+1) of every q and k head
// are rotated by pos * theta^(-2p/hd), pos = position in the sequence; the backward pass applies the transpose.
// The angles' cosines and sines come from a table [s][hd/2] of (cos, sin), built once in double precision.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rope_table_kernel(float2* table, int s, int half, double theta) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)s * half) return;
  const int pos = (int)(i / half), p = (int)(i % half);
  const double ang = (double)pos * pow(theta, -(double)p / (double)half);
  table[i] = make_float2((float)cos(ang), (float)sin(ang));
}

// in place on the first nh heads of every row of x [rows, ld]; one 16-byte vector per thread and step
template <typename T>
__global__ __launch_bounds__(256) void rope_kernel(T* x, int64_t ld, int64_t rows, int s, int nh, int hd, const float2* table,
                                                   int inverse) {
  constexpr int V = Vec<T>::N;
  const int per_row = nh * hd / V, vec_per_head = hd / V;
  const int64_t total = rows * per_row;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t row = i / per_row;
    const int c = (int)(i % per_row);
    const int pos = (int)(row % s), p0 = (c % vec_per_head) * (V / 2);          // first pair index inside the head
    T* ptr = x + row * ld + (int64_t)c * V;
    Vec<T> v = ldv(ptr);
    const float2* t = table + (int64_t)pos * (hd / 2) + p0;
#pragma unroll
    for (int q = 0; q < V / 2; ++q) {
      const float2 cs = t[q];
      const float sn = inverse ? -cs.y : cs.y;
      const float a = to_f32(v.v[2 * q]), b = to_f32(v.v[2 * q + 1]);
      v.v[2 * q] = from_f32<T>(a * cs.x - b * sn);
      v.v[2 * q + 1] = from_f32<T>(a * sn + b * cs.x);
    }
    stv(ptr, v);
  }
}

hipError_t rope_table(float* table, int s, int hd, double theta, hipStream_t st) {
  if (s < 1 || hd < 2 || hd % 2 || !(theta > 0.0) || !table) return hipErrorInvalidValue;
  const int64_t n = (int64_t)s * (hd / 2);
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (float2*)table, s, hd / 2, theta);
  return hipGetLastError();
}

hipError_t rope_apply(DType dt, void* x, int64_t ld, int64_t rows, int s, int nh, int hd, const float* table, int inverse,
                      hipStream_t st) {
  const int V = dt == DT_F32 ? 4 : 8;
  if (rows < 1 || s < 1 || nh < 1 || hd % V || ld % V || !x || !table || ((uintptr_t)x & 15)) return hipErrorInvalidValue;
  const int64_t total = rows * (nh * hd / V), want = (total + 255) / 256;
  const int grid = (int)(want > 16384 ? 16384 : want);
  if (dt == DT_F32) hipLaunchKernelGGL((rope_kernel<float>), dim3(grid), dim3(256), 0, st, (float*)x, ld, rows, s, nh, hd, (const float2*)table, inverse);
  else hipLaunchKernelGGL((rope_kernel<bf16>), dim3(grid), dim3(256), 0, st, (bf16*)x, ld, rows, s, nh, hd, (const float2*)table, inverse);
  return hipGetLastError();
}

}  // namespace stg
