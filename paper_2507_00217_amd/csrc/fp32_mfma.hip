// fp32 matrix products and attention on the fp32 matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 products and
// sums), the compute path of the fp32 configuration.
//
// What bounds it: the stages that run in fp32 are small (a schedule is checked on them), so a product has far fewer
// 64 x 64 output tiles than the chip has CUs and what counts is the length of the serial chain in one workgroup, not the
// matrix rate.  So the wavefronts of a workgroup share one output tile and split the REDUCTION between them (each takes
// every W-th slice of it), and the partial tiles are added up through LDS in wavefront order at the end: no barrier inside
// the loop, no workspace, the same bits on every run.  Operand fragments go global -> registers directly (but for 32 x 32 tiles): an fp32 MFMA
// takes 32 cycles, so a 64 x 64 wavefront tile asks for 16 bytes per clock and CU, a quarter of what the caches deliver,
// and staging tiles in LDS would buy nothing but barriers.  The order of the reduction inside a 16-deep slice is free as
// long as both operands agree: lane group g takes k = 4g .. 4g + 3 in the four MFMAs of a slice, so an operand whose
// reduction index is contiguous is read 16 bytes per lane; an operand whose reduction index is the slow one is read
// row by row, NB consecutive columns per lane, which become column c of NB different 16 x 16 blocks (block j's column c
// is column NB * c + j of the tile).
//
// Measured, a two-layer stage of 128 x 256 tokens x width and four microbatches: 6918 us with the plain kernels, whose
// products ran in 8 workgroups with one thread walking all of K (107 us each, 5 us now); a Llama-style layer of 448 x 512: 4563
// us before.  Products that fill the chip reach 113-123 of the 152 TFLOP/s a large library product does (1400 x 8192 x 1024).
#include "common.h"
#include <type_traits>

namespace stg {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

namespace {

enum Epi32 { E32_GENERAL = 0, E32_GELU = 1, E32_SWIGLU = 2, E32_DGELU = 3, E32_DSWIGLU = 4 };

constexpr unsigned OOB32 = 0x80000000u;      // a buffer load at or past num_records returns zeros

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// N consecutive floats at byte offset `off`; past the end of the buffer: zeros
template <int N> __device__ __forceinline__ void ld_buf(float (&v)[N], __amdgpu_buffer_rsrc_t rs, unsigned off) {
  if constexpr (N == 4) {
    const f32x4 t = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = t[i];
  } else if constexpr (N == 2) {
    const f32x2 t = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0));
    v[0] = t[0]; v[1] = t[1];
  } else {
    v[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0));
  }
}

// One operand of a wavefront's tile: NB blocks of 16 rows (of C for A, columns of C for B).
// KC: reduction index contiguous in memory; block i's row c is row row0 + 16 * i + c.
// else: reduction index slow; block i's row c is row row0 + SP * c + i % SP (+ `second` rows for the blocks from SP on, where
// SP = NB, or NB / 2 when the tile is a SwiGLU one and its upper blocks are the `up` columns of the same features).
template <bool KC, int NB, int SP>
struct Operand {
  __amdgpu_buffer_rsrc_t rs;
  unsigned base[KC ? NB : NB / SP];
  unsigned ld4;                        // bytes per row of the matrix in memory
  int K;
  __device__ __forceinline__ void init(const void* p, int64_t ld, int row0, int rows, int Kred, int second, int c, int g) {
    const int64_t span = KC ? (int64_t)((second ? 2 * rows : rows) - 1) * ld + Kred : (int64_t)(Kred - 1) * ld + (second ? second + rows : rows);
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (unsigned)(span * 4), 0x00020000);
    ld4 = (unsigned)(ld * 4); K = Kred;
    if (KC) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int r = row0 + 16 * i + c;
        base[i] = r < rows ? (unsigned)r * ld4 + (unsigned)g * 16u : OOB32;
      }
    } else {
#pragma unroll
      for (int h = 0; h < NB / SP; ++h) {
        const int r = row0 + SP * c;
        base[h] = r < rows ? (unsigned)(r + h * second) * 4u + (unsigned)(4 * g) * ld4 : OOB32;
      }
    }
  }
  // fragments of the slice k .. k + 15: f[i][j] is what MFMA j of block i takes from this lane.  Slices past the end read zeros.
  __device__ __forceinline__ void load(f32x4 (&f)[NB], int k, int g) const {
    if (KC) {
      const bool in = k + 4 * g < K;                                    // K % 4 == 0
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        float v[4];
        ld_buf<4>(v, rs, in ? base[i] + (unsigned)k * 4u : OOB32);
#pragma unroll
        for (int j = 0; j < 4; ++j) f[i][j] = v[j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int h = 0; h < NB / SP; ++h) {
          float v[SP];
          ld_buf<SP>(v, rs, base[h] + (unsigned)(k + j) * ld4);          // rows >= K lie past the end of the buffer
#pragma unroll
          for (int i = 0; i < SP; ++i) f[h * SP + i][j] = v[i];
        }
    }
  }
};

__device__ __forceinline__ float gelu32(float u) { return 0.5f * u * (1.f + erff(u * 0.70710678118654752f)); }
__device__ __forceinline__ float dgelu32(float u) {
  return 0.5f * (1.f + erff(u * 0.70710678118654752f)) + u * 0.39894228040143268f * __expf(-0.5f * u * u);
}
__device__ __forceinline__ float sigm32(float v) { return 1.f / (1.f + __expf(-v)); }

// ---- operands through LDS ----------------------------------------------------------------------------------------------
// Fragments loaded straight into registers are 16 rows x 64 bytes at a time where the reduction is contiguous, half of every
// line, which a CU takes at 30 bytes a clock: the matrix cores wait.  Here a wavefront's slice is 32 deep, whole lines, and goes
// through a place of its own in LDS: nobody else reads it, so there is no barrier.  Once its fragments are in registers the next
// slice is on its way there; it has this slice's 32 MFMAs, and those of the other wavefronts of the SIMD, to land.  64 KiB for eight
// wavefronts, two workgroups per CU.  (Two places per wavefront, one workgroup per CU: 448 x 512 x 2816 16.6 us instead of 15.5, 700 x 1024 x
// 3072 52 instead of 43.)
//   reduction contiguous: [32 rows][8 pieces of 16 bytes], piece p of row r in place p ^ ((r >> 1) & 7): 16 lanes read the same
//     piece of 16 rows, from all banks
//   reduction slow: [32 reduction rows][8 pieces = 32 columns], row k in place k ^ ((k >> 2) & 1), piece p in p ^ (((k >> 3) & 1) << 2):
//     the four lane groups read rows 4 apart, from different banks
typedef __attribute__((address_space(3))) char lds_char;
typedef int rsrc32 __attribute__((ext_vector_type(4)));
constexpr int SLICE32 = 32, SLICE_BYTES = 32 * SLICE32 * 4, SLICE_LOADS = SLICE_BYTES / 1024;      // per operand

template <bool KC, bool GLU>
struct SliceLoad {
  rsrc32 rs;
  unsigned off[SLICE_LOADS], ld4;
  int kp, K;
  __device__ __forceinline__ void init(const void* p, int64_t ld, int row0, int rows, int Kred, int second, int lane) {
    const uint64_t a = (uint64_t)p;
    const int64_t span = KC ? (int64_t)(rows - 1) * ld + Kred : (int64_t)(Kred - 1) * ld + (second ? second + rows : rows);
    rs = rsrc32{(int)(unsigned)a, (int)(unsigned)((a >> 32) & 0xffffu), (int)(unsigned)(span * 4), 0x00020000};
    ld4 = (unsigned)(ld * 4); K = Kred;
#pragma unroll
    for (int j = 0; j < SLICE_LOADS; ++j) {
      const int x = j * 8 + (lane >> 3);                                          // place of the row
      if (KC) {
        const int pc = (lane & 7) ^ ((x >> 1) & 7);
        if (j == 0) kp = pc * 4;                                                  // (rows 8 apart: piece ^ 4)
        off[j] = row0 + x < rows ? (unsigned)(row0 + x) * ld4 + (unsigned)pc * 16u : OOB32;
      } else {
        const int k = x ^ ((x >> 2) & 1), pc = (lane & 7) ^ (((k >> 3) & 1) << 2), col = row0 + (GLU ? pc & 3 : pc) * 4;
        off[j] = col < rows ? (unsigned)(col + (GLU && pc > 3 ? second : 0)) * 4u + (unsigned)k * ld4 : OOB32;
      }
    }
  }
  __device__ __forceinline__ void load(lds_char* dst, int k0) const {
#pragma unroll
    for (int j = 0; j < SLICE_LOADS; ++j) {
      // past the end of the reduction: contiguous pieces are redirected, rows of a slow one lie past the end of the buffer
      const unsigned o = KC ? (k0 + (kp ^ ((j & 1) << 4)) < K ? off[j] + (unsigned)k0 * 4u : OOB32) : off[j] + (unsigned)k0 * ld4;
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"((unsigned)(size_t)(dst + j * 1024)), "v"(o), "s"(rs) : "memory");
    }
  }
};

template <bool BKC, int W, bool GLU>
__device__ __forceinline__ void reduce_via_lds(f32x4 (&acc)[2][2], const GemmArgs& g, int m0, int n0, int nfeat, lds_char* ring, int w, int lane) {
  typedef __attribute__((address_space(3))) const f32x4* p4;
  typedef __attribute__((address_space(3))) const f32x2* p2;
  typedef __attribute__((address_space(3))) const float* p1;
  const int c = lane & 15, gr = lane >> 4;
  SliceLoad<true, false> la; SliceLoad<BKC, GLU> lb;
  la.init(g.A, g.lda, m0, g.M, g.K, 0, lane);
  lb.init(g.B, g.ldb, n0, nfeat, g.K, GLU ? nfeat : 0, lane);
  lds_char* mine = ring + w * (2 * SLICE_BYTES);
  auto fetch = [&](int k) { la.load(mine, k); lb.load(mine + SLICE_BYTES, k); };
  // fragments: h = 16-deep half, f[h][block][j] as in Operand
  auto read_kc = [&](f32x4 (&f)[2][2], lds_char* st) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i) f[h][i] = *(p4)(st + (16 * i + c) * 128 + (((4 * h + gr) ^ ((c >> 1) & 7)) << 4));
  };
  auto read_slow = [&](f32x4 (&f)[2][2], lds_char* st, auto glu) __attribute__((always_inline)) {
    const int x = (gr >> 1) << 2;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        lds_char* row = st + (16 * h + 4 * gr + (j ^ (gr & 1))) * 128;
        if constexpr (decltype(glu)::value) {
          f[h][0][j] = *(p1)(row + (((c >> 2) ^ x) << 4) + (c & 3) * 4);
          f[h][1][j] = *(p1)(row + ((((c >> 2) + 4) ^ x) << 4) + (c & 3) * 4);
        } else {
          const f32x2 v = *(p2)(row + (((c >> 1) ^ x) << 4) + (c & 1) * 8);
          f[h][0][j] = v[0]; f[h][1][j] = v[1];
        }
      }
  };
  // The halves of the slices are summed apart: the rounding errors of a sum grow with its length, and eight wavefronts with one sum
  // each were up to 1.36 times as far from 64 bits as the sixteen of a 16 x 16 tile (input gradients 214 x 576 x 2720 3.4e-7, 2.5e-7).
  f32x4 odd[2][2] = {};
  const int step = W * SLICE32;
  if (w * SLICE32 < g.K) fetch(w * SLICE32);
  for (int k = w * SLICE32; k < g.K; k += step) {
    __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0): the slice has landed
    asm volatile("" ::: "memory");
    f32x4 fa[2][2], fb[2][2];
    read_kc(fa, mine);
    if constexpr (BKC) read_kc(fb, mine + SLICE_BYTES); else read_slow(fb, mine + SLICE_BYTES, std::integral_constant<bool, GLU>{});
    __builtin_amdgcn_s_waitcnt(0xc07f);                  // lgkmcnt(0): the fragments are in registers, the place is free
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (k + step < g.K) fetch(k + step);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int n = 0; n < 2; ++n) {
            f32x4& s = h ? odd[i][n] : acc[i][n];
            s = mfma4(fb[h][n][j], fa[h][i][j], s);
          }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int n = 0; n < 2; ++n) acc[i][n] += odd[i][n];
}

// The tile at (m0, n0), 16 * MB x 16 * NB outputs (SwiGLU forward: 8 * NB features, gate and up), by W wavefronts that split
// the reduction.  The MFMA is issued with the operands swapped, which leaves every lane with columns of one row of C.
// `red`: W * MB * NB * 64 float4 of LDS.  nseg > 1 (weight gradients): the product of the operand pair moved by seg_delta[s]
// bytes is added to C for s = 0, 1, ... in turn -- the same bits as one launch per pair.
// VIA_LDS: the operands of a 32 x 32 tile go through LDS first (`red` serves as the ring).
template <int MODE, int MB, int NB, int W, int EPI, bool VIA_LDS = false>
__device__ __forceinline__ void tile32(const GemmArgs& g, int m0, int n0, f32x4* red, int nseg, const int64_t* seg_delta) {
  constexpr bool AKC = MODE != GEMM_TN, BKC = MODE == GEMM_NT, GLU = EPI == E32_SWIGLU;
  static_assert(!GLU || (!BKC && NB >= 2), "gate and up blocks");
  constexpr int U = MB * NB >= 4 ? 1 : 2;              // 16-deep slices fetched at a time
  constexpr int SPB = GLU ? NB / 2 : NB;               // consecutive columns per lane of a slow-index B
  constexpr int NQ = MB * NB;                          // 4-column pieces of the tile per lane
  const int lane = threadIdx.x & 63, c = lane & 15, gr = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nfeat = GLU ? g.N / 2 : g.N;
  f32x4 run[(NQ + W - 1) / W];                         // weight gradients over several segments: C so far

  for (int sg = 0; sg < nseg; ++sg) {
    f32x4 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t delta = MODE == GEMM_TN && sg > 0 ? seg_delta[sg] : 0;
    if constexpr (VIA_LDS) {
      reduce_via_lds<BKC, W, GLU>(acc, g, m0, n0, nfeat, (lds_char*)red, w, lane);
      __syncthreads();                                 // the ring becomes `red`
    } else {
    Operand<AKC, MB, MB> oa; Operand<BKC, NB, SPB> ob;
    oa.init((const char*)g.A + delta, g.lda, m0, g.M, g.K, 0, c, gr);
    ob.init((const char*)g.B + delta, g.ldb, n0, nfeat, g.K, GLU ? nfeat : 0, c, gr);
    f32x4 fa[2][U][MB], fb[2][U][NB];
    auto load = [&](int set, int ch) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        oa.load(fa[set][u], (ch * U + u) * 16, gr);
        ob.load(fb[set][u], (ch * U + u) * 16, gr);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](int set) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[i][n] = mfma4(fb[set][u][n][j], fa[set][u][i][j], acc[i][n]);
      __builtin_amdgcn_sched_barrier(0);
    };
    // wavefront w takes slices w, w + W, ...; the next one is always in flight (past the end it reads zeros without
    // touching memory, which keeps the loop free of branches around loads)
    const int nch = (g.K + 16 * U - 1) / (16 * U);
    load(0, w);
    for (int ch = w; ch < nch; ch += 2 * W) {
      load(1, ch + W);
      mul(0);
      load(0, ch + 2 * W);
      mul(1);
    }
    }
    if (sg > 0) __syncthreads();                       // the previous segment's partial tiles have been read
    // quad q = i * NB + p of a lane: row i of its row blocks, 4 consecutive columns (see quad_n below)
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int p = 0; p < NB; ++p) {
        f32x4 v;
        if constexpr (BKC || SPB == 1) v = acc[i][p];
        else if constexpr (SPB == 4) v = f32x4{acc[i][0][p], acc[i][1][p], acc[i][2][p], acc[i][3][p]};
        else {                                         // SPB == 2: half = which pair of blocks, e = which pair of rows
          const int half = p / 2, e = (p % 2) * 2;
          v = f32x4{acc[i][2 * half][e], acc[i][2 * half + 1][e], acc[i][2 * half][e + 1], acc[i][2 * half + 1][e + 1]};
        }
        red[(w * NQ + i * NB + p) * 64 + lane] = v;
      }
    __syncthreads();
    if (MODE == GEMM_TN) {
#pragma unroll
      for (int t = 0; t < (NQ + W - 1) / W; ++t) {
        const int q = w + t * W;
        if (q >= NQ) break;
        const int i = q / NB, p = q % NB;
        const int m = m0 + MB * c + i, n = n0 + (NB == 4 ? 16 * gr + 4 * p : NB == 2 ? 8 * gr + 4 * p : 4 * gr);
        f32x4 v = red[q * 64 + lane];
#pragma unroll
        for (int ww = 1; ww < W; ++ww) v += red[(ww * NQ + q) * 64 + lane];
        if (m < g.M && n < g.N) {
          f32x4* C = reinterpret_cast<f32x4*>((float*)g.C + (int64_t)m * g.ldc + n);
          run[t] = (sg == 0 ? *C : run[t]) + v;
          if (sg == nseg - 1) *C = run[t];
        }
      }
    }
  }
  if (MODE == GEMM_TN) return;

  auto sum = [&](int q) __attribute__((always_inline)) {
    f32x4 v = red[q * 64 + lane];
#pragma unroll
    for (int ww = 1; ww < W; ++ww) v += red[(ww * NQ + q) * 64 + lane];
    return v;
  };
  constexpr int NQE = GLU ? NQ / 2 : NQ;               // SwiGLU: a gate quad and the up quad of the same features together
#pragma unroll
  for (int t = 0; t < (NQE + W - 1) / W; ++t) {
    const int qe = w + t * W;
    if (qe >= NQE) break;
    const int i = GLU ? qe / (NB / 2) : qe / NB, p = GLU ? qe % (NB / 2) : qe % NB;
    const int m = m0 + 16 * i + c;
    const int n = n0 + (BKC ? 16 * p + 4 * gr : SPB == 4 ? 16 * gr + 4 * p : SPB == 2 ? 8 * gr + 4 * p : 4 * gr);
    f32x4 v = sum(i * NB + p);
    if (GLU) {
      f32x4 up = sum(i * NB + p + NB / 2);
      if (m < g.M && n < nfeat) {
        if (g.bias) { v += *reinterpret_cast<const f32x4*>((const float*)g.bias + n); up += *reinterpret_cast<const f32x4*>((const float*)g.bias + nfeat + n); }
        float* z = (float*)g.C + (int64_t)m * g.ldc + n;
        *reinterpret_cast<f32x4*>(z) = v;
        *reinterpret_cast<f32x4*>(z + nfeat) = up;
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = v[e] * sigm32(v[e]) * up[e];
        *reinterpret_cast<f32x4*>((float*)g.C2 + (int64_t)m * g.ldc2 + n) = o;
      }
      continue;
    }
    if (m >= g.M || n >= g.N) continue;
    if (EPI == E32_DGELU || EPI == E32_DSWIGLU) {
      float* z = (float*)g.Z + (int64_t)m * g.ldz + n;
      f32x4 a = *reinterpret_cast<f32x4*>(z);
      if (g.C) *reinterpret_cast<f32x4*>((float*)g.C + (int64_t)m * g.ldc + n) = v;
      if (EPI == E32_DGELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = v[e] * dgelu32(a[e]);
        *reinterpret_cast<f32x4*>(z) = a;
      } else {
        f32x4 u = *reinterpret_cast<f32x4*>(z + g.N);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gv = a[e], sg = sigm32(gv);
          a[e] = v[e] * u[e] * (sg + gv * sg * (1.f - sg));
          u[e] = v[e] * gv * sg;
        }
        *reinterpret_cast<f32x4*>(z) = a;
        *reinterpret_cast<f32x4*>(z + g.N) = u;
      }
      continue;
    }
    if (g.bias) v += *reinterpret_cast<const f32x4*>((const float*)g.bias + n);
    if (g.R) v += *reinterpret_cast<const f32x4*>((const float*)g.R + (int64_t)m * g.ldr + n);
    *reinterpret_cast<f32x4*>((float*)g.C + (int64_t)m * g.ldc + n) = v;
    if (EPI == E32_GELU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gelu32(v[e]);
      *reinterpret_cast<f32x4*>((float*)g.C2 + (int64_t)m * g.ldc2 + n) = v;
    }
  }
}

// tile `idx` of the walk order: groups of 8 tile rows, column by column inside a group
__device__ __forceinline__ void tile32_of(int idx, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int in_group = 8 * tiles_n, gid = idx / in_group, first = gid * 8, gsz = min(tiles_m - first, 8);
  tm = first + (idx % in_group) % gsz;
  tn = (idx % in_group) / gsz;
}

template <int MODE, int MB, int NB, int W, int EPI, bool VIA_LDS>
__global__ __launch_bounds__(W * 64) void gemm32_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  static_assert(!VIA_LDS || (MB == 2 && NB == 2), "32 x 32 tiles; their partial tiles take half of the ring");
  __shared__ __attribute__((aligned(1024))) f32x4 red[VIA_LDS ? W * 2 * SLICE_BYTES / 16 : W * MB * NB * 64];
  int tm, tn;
  tile32_of(blockIdx.x, tiles_m, tiles_n, tm, tn);
  tile32<MODE, MB, NB, W, EPI, VIA_LDS>(g, tm * 16 * MB, tn * (EPI == E32_SWIGLU ? 8 : 16) * NB, red, 1, nullptr);
}

// several weight-gradient products in one launch, one workgroup per tile of the concatenated tile list
constexpr int GROUP32_MAX = 8;
struct Wgrad32 { const void *A, *B; void* C; int64_t lda, ldb, ldc; int M, N, K, first; };
struct Wgrad32Group { int n, nseg; int64_t seg_delta[GEMM_MAX_SEG]; Wgrad32 p[GROUP32_MAX]; };

template <int MB, int NB, int W>
__global__ __launch_bounds__(W * 64) void wgrad32_group_kernel(Wgrad32Group gg) {
  __shared__ f32x4 red[W * MB * NB * 64];
  int pi = 0;
  while (pi + 1 < gg.n && (int)blockIdx.x >= gg.p[pi + 1].first) ++pi;
  const Wgrad32& p = gg.p[pi];
  GemmArgs g{};
  g.M = p.M; g.N = p.N; g.K = p.K; g.A = p.A; g.lda = p.lda; g.B = p.B; g.ldb = p.ldb; g.C = p.C; g.ldc = p.ldc;
  int tm, tn;
  tile32_of((int)blockIdx.x - p.first, (g.M + 16 * MB - 1) / (16 * MB), (g.N + 16 * NB - 1) / (16 * NB), tm, tn);
  tile32<GEMM_TN, MB, NB, W, E32_GENERAL>(g, tm * 16 * MB, tn * 16 * NB, red, gg.nseg, gg.seg_delta);
}

// Tile shapes: 0 = 64 x 64 by 4 wavefronts, 1 = 32 x 32 by 8, 2 = 16 x 16 (SwiGLU forward: 16 x 32) by 16.  The rule takes
// the one whose matrix-core time on the fullest CU is least: rounds of one tile per CU, times the tile's area, times what
// the shape loses to operand traffic.  For 32 x 32 tiles that depends on their form (via_lds32): 1.2 with a slow-index B, straight to registers
// or through LDS (against 64 x 64 1.2 to 1.28 and 1.2 to 1.28 over 1024 x 2432 .. 1400 x 4096, K 448 .. 1024; SwiGLU 1.2 to 1.55: 1084 x 2016 x 448 54.8 us in
// 64 x 64, 62.3, 900 x 1300 x 640 44.3, 52.8), 1.45 with both operands reduction-contiguous straight to registers and 1.19 through LDS
// (1024 x 2432 x 1024 56.8 / 55.1, GELU backward 900 x 2600 x 640 55.0 / 44.4, 700 x 1024 x 1024 20.9 / 18.6), counted in pairs of rounds on wide
// outputs, whose two workgroups per CU share less (171 x 4000 x 1024 20.9 / 24.3, 222 x 3232 x 512 12.6 / 14.4, 1084 x 4032 x 448 51.8 / 53.5).  M 1400, N 8192, K 1024: 208 /
// 234 / 507 us with a slow-index B.  The rounds decide where a shape does not fill the chip (448 x 512 x 1408: 26.1 / 9.2 / 18.2 us, 128 x 256 x 1024:
// 19.9 / 7.2 / 4.8 us).
int pick32(int mode, int M, int N, bool via_lds) {
  const double loss[3] = {1., mode != GEMM_NT ? 1.2 : via_lds ? 1.19 : 1.45, mode != GEMM_NT ? 2.4 : 2.8};
  static const int tile[3] = {64, 32, 16};
  const int n_cu = cu_count();
  int best = 0;
  double bt = 0.;
  for (int i = 0; i < 3; ++i) {
    const int64_t tiles = (int64_t)((M + tile[i] - 1) / tile[i]) * ((N + tile[i] - 1) / tile[i]);
    int64_t rounds = (tiles + n_cu - 1) / n_cu;
    if (i == 1 && mode == GEMM_NT && via_lds && N > 2048 && rounds > 1) rounds += rounds & 1;
    const double t = (double)rounds * tile[i] * tile[i] * loss[i];
    if (i == 0 || t < bt) { best = i; bt = t; }
  }
  return best;
}

// Whether the operands of 32 x 32 tiles go through LDS (us, straight to registers / through LDS: input gradients 448 x 512 x 512 6.2 / 5.1, x
// 1536 13.8 / 10.0, x 2816 22.8 / 15.8, 700 x 1024 x 3072 66 / 44, forward 448 x 512 x 1408 11.3 / 9.2, 700 x 3072 x 1024 54.5 / 50.4, SwiGLU 300 x 1024 x 768
// 20.6 / 16.7, its backward 448 x 1408 x 512 15.7 / 13.2).  Not where
//  - rows do not start on 128-byte lines, so that a slice's rows are not whole lines, unless the reduction is long (forward 700 x 1024 x 264
//    7.3 / 8.8, 1000 x 1000 x 520 13.2 / 14.9, x 1288 31.7 / 30.7; GELU backward 700 x 1024 x 504 11.3 / 14.2, x 1288 28.2 / 27.6;
//    SwiGLU 114 x 1020 x 1024 12.0 / 12.9);
//  - there are more tiles than the two per CU that its LDS lets in at once, where four of the other form are, and little to win: up to
//    256 terms (forward 700 x 1024 x 256 7.6 / 8.1, GELU backward 9.7 / 11.0, but input gradients 8.5 / 7.9), forward of more than four
//    tiles per CU up to 512 (448 x 2816 x 512 18.1 / 20.6), GELU (222 x 3232 x 416 12.5 / 13.8, 700 x 1024 x 1408 27.8 / 29.7), SwiGLU of more than four
//    (448 x 1408 x 512 22.7 / 23.2); and SwiGLU up to 256 terms at any count (514 x 432 x 64 4.2 / 4.4, 374 x 464 x 256 5.6 / 5.9).
template <int MODE, int EPI>
bool via_lds32(const GemmArgs& g) {
  constexpr bool BKC = MODE == GEMM_NT;
  const int64_t tiles = (int64_t)((g.M + 31) / 32) * ((g.N + 31) / 32), n_cu = cu_count();
  const bool lines = g.lda % 32 == 0 && g.ldb % 32 == 0 && (((uintptr_t)g.A | (uintptr_t)g.B) & 127) == 0;
  if (EPI == E32_GELU && tiles > 2 * n_cu) return false;
  if (EPI == E32_SWIGLU && (tiles > 4 * n_cu || g.K <= 256)) return false;
  if (!lines) return g.K >= 1280;
  if (EPI == E32_GENERAL && BKC) return tiles <= 2 * n_cu || g.K > 64;
  return tiles <= 2 * n_cu || g.K > (EPI == E32_GENERAL && tiles > 4 * n_cu ? 512 : 256);
}

template <int MODE, int MB, int NB, int W, int EPI, bool VIA_LDS = false>
hipError_t launch32(const GemmArgs& g, hipStream_t s) {
  constexpr int TM = 16 * MB, TN = (EPI == E32_SWIGLU ? 8 : 16) * NB;
  const int tiles_m = (g.M + TM - 1) / TM, tiles_n = ((EPI == E32_SWIGLU ? g.N / 2 : g.N) + TN - 1) / TN;
  hipLaunchKernelGGL((gemm32_kernel<MODE, MB, NB, W, EPI, VIA_LDS>), dim3(tiles_m * tiles_n), dim3(W * 64), 0, s, g, tiles_m, tiles_n);
  return hipGetLastError();
}
template <int MODE, int EPI>
hipError_t pick_launch32(const GemmArgs& g, hipStream_t s, int shape) {
  constexpr int NB3 = EPI == E32_SWIGLU ? 2 : 1;
  // (a forced shape keeps to LDS on fewer conditions, so that tests reach it at the edges of its slices)
  const bool via_lds = shape > 0 ? !((EPI == E32_GELU || EPI == E32_SWIGLU) && (int64_t)((g.M + 31) / 32) * ((g.N + 31) / 32) > 4 * cu_count()) : via_lds32<MODE, EPI>(g);
  const int which = shape > 0 ? shape - 1 : pick32(MODE, g.M, g.N, via_lds);
  if (which == 0) return launch32<MODE, 4, 4, 4, EPI>(g, s);
  if (which == 1) return via_lds ? launch32<MODE, 2, 2, 8, EPI, true>(g, s) : launch32<MODE, 2, 2, 8, EPI>(g, s);
  return launch32<MODE, 1, NB3, 16, EPI>(g, s);
}

}  // namespace

bool gemm32_supported(const GemmArgs& g) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
  auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  if (!al16(g.A) || !al16(g.B) || !al16(g.C) || !al16(g.R) || !al16(g.bias)) return false;
  if (g.lda % 4 || g.ldb % 4 || g.ldc % 4 || (g.R && g.ldr % 4) || g.N % 4) return false;
  if (g.mode != GEMM_TN && g.K % 4) return false;
  if (g.mode == GEMM_TN && g.M % 4) return false;
  if ((g.mode == GEMM_TN) != (g.acc_f32 != 0) || (g.acc_f32 && (g.R || g.bias))) return false;
  // an operand with a slow reduction index relies on its rows past K lying past the end of its buffer: no row may overlap the next
  if (g.lda < (g.mode == GEMM_TN ? g.M : 0) || g.ldb < (g.mode == GEMM_NT ? 0 : g.N)) return false;
  // Short reductions over large outputs move C and little else, which the plain kernel's many small workgroups do better than workgroups
  // with 64 KiB of LDS (us, plain / these: weight gradients 2048 x 2048 x 52 17.9 / 19.2, x 64 18.3 / 19.1, x 80 20.5 / 19.3; 4096 x 4096 x 43
  // 47 / 63; 1024 x 1024 x 32 8.7 / 7.0; forward 4096 x 4096 x 48 41 / 56, input gradients 42 / 52).
  if (g.K <= 64 && !g.act && !g.act_bwd && (int64_t)((g.M + 63) / 64) * ((g.N + 63) / 64) >= 4 * cu_count()) return false;
  const int64_t lim = (int64_t)1 << 29;        // byte offsets stay below 2 GiB, slices fetched past the end (less than 2048 rows) included
  const int64_t a_rows = g.mode == GEMM_TN ? g.K + 2048 : g.M, b_rows = g.mode == GEMM_NT ? g.N : (int64_t)g.K + 2048;
  if (a_rows * g.lda >= lim || b_rows * g.ldb >= lim || (g.mode != GEMM_TN && (int64_t)g.K + 2048 >= lim)) return false;
  if (g.act && (g.mode != GEMM_NN || g.R || (g.act != 1 && g.act != 2) || !al16(g.C2) || g.ldc2 % 4 || (g.act == 2 && g.N % 8))) return false;
  if (g.act_bwd && (g.mode != GEMM_NT || g.act || g.R || g.bias || (g.act_bwd != 1 && g.act_bwd != 2) || !al16(g.Z) || g.ldz % 4)) return false;
  return true;
}

hipError_t gemm32(const GemmArgs& g, hipStream_t s, int shape) {
  switch (g.mode) {
    case GEMM_NN:
      if (g.act == 1) return pick_launch32<GEMM_NN, E32_GELU>(g, s, shape);
      if (g.act == 2) return pick_launch32<GEMM_NN, E32_SWIGLU>(g, s, shape);
      return pick_launch32<GEMM_NN, E32_GENERAL>(g, s, shape);
    case GEMM_NT:
      if (g.act_bwd == 1) return pick_launch32<GEMM_NT, E32_DGELU>(g, s, shape);
      if (g.act_bwd == 2) return pick_launch32<GEMM_NT, E32_DSWIGLU>(g, s, shape);
      return pick_launch32<GEMM_NT, E32_GENERAL>(g, s, shape);
    case GEMM_TN: return wgrad32_group(&g, 1, 1, nullptr, s, shape);
  }
  return hipErrorInvalidValue;
}

bool wgrad32_group_supported(const GemmArgs* list, int n, int nseg, const int64_t* seg_delta) {
  if (n < 1 || nseg < 1 || nseg > GEMM_MAX_SEG || (nseg > 1 && !seg_delta)) return false;
  for (int s = 1; s < nseg; ++s)
    if (seg_delta[s] % 16) return false;
  for (int i = 0; i < n; ++i)
    if (list[i].mode != GEMM_TN || !gemm32_supported(list[i])) return false;
  return true;
}

// One tile shape for the whole list, by the rule above on the list's tiles; both shapes split the reduction over four wavefronts
// in the same slices, so a product's bits depend neither on the shape nor on what it is grouped with.  Four products of 448
// tokens x 512 .. 2816: 44 us with eight wavefronts per 32 x 32 tile, 41 with four, 46 in 64 x 64 tiles (two to a CU: a round and a
// half); two layers of 128 tokens x 256 .. 1024: 16.5, 12.0 and 13.5.
hipError_t wgrad32_group(const GemmArgs* list, int n, int nseg, const int64_t* seg_delta, hipStream_t s, int shape) {
  const int n_cu = cu_count();
  int64_t area[2] = {0, 0};
  for (int which = 0; which < 2; ++which) {
    const int t = which == 0 ? 64 : 32;
    for (int i = 0; i < n; ++i) area[which] += (int64_t)((list[i].M + t - 1) / t) * ((list[i].N + t - 1) / t);
    area[which] = (area[which] + n_cu - 1) / n_cu * t * t;
  }
  const bool wide = shape > 0 ? shape == 1 : (double)area[0] <= 1.2 * (double)area[1];
  const int t = wide ? 64 : 32;
  for (int i0 = 0; i0 < n; i0 += GROUP32_MAX) {
    Wgrad32Group gg;
    gg.n = n - i0 < GROUP32_MAX ? n - i0 : GROUP32_MAX; gg.nseg = nseg;
    for (int i = 0; i < GEMM_MAX_SEG; ++i) gg.seg_delta[i] = i > 0 && i < nseg ? seg_delta[i] : 0;
    int total = 0;
    for (int i = 0; i < gg.n; ++i) {
      const GemmArgs& a = list[i0 + i];
      gg.p[i] = Wgrad32{a.A, a.B, a.C, a.lda, a.ldb, a.ldc, a.M, a.N, a.K, total};
      total += ((a.M + t - 1) / t) * ((a.N + t - 1) / t);
    }
    if (wide) hipLaunchKernelGGL((wgrad32_group_kernel<4, 4, 4>), dim3(total), dim3(256), 0, s, gg);
    else hipLaunchKernelGGL((wgrad32_group_kernel<2, 2, 4>), dim3(total), dim3(256), 0, s, gg);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Attention.  One workgroup per 16 queries (forward, dQ) or 16 keys (dK/dV) of a head; its W wavefronts take every W-th
// block of 16 keys (queries) and are merged through LDS in wavefront order at the end, so that short sequences and few heads
// still spread over the chip and no wavefront has a long serial chain.  Everything is computed transposed: the scores of a
// block leave MFMA as D[key][query] with lane (c, g) holding query c and keys 4g .. 4g + 3, which is exactly what the next
// product wants as its B operand -- probabilities never leave their registers.
// ---------------------------------------------------------------------------
namespace {

constexpr int AW = 8;                 // wavefronts per workgroup

// fragment of 16 rows (row index `row` for this lane) x HD, reduction along HD: t-th float4 at 16 t + 4 g
template <int HD> __device__ __forceinline__ void ld_rows(f32x4 (&f)[HD / 16], const float* row, int g) {
#pragma unroll
  for (int t = 0; t < HD / 16; ++t) f[t] = *reinterpret_cast<const f32x4*>(row + 16 * t + 4 * g);
}
// fragment with the reduction along the 16 rows: rows r0 + 4 g + j (clamped to the last one), HD / 16 consecutive columns from
// (HD / 16) * c on; f[j][i]: block i, MFMA j
template <int HD> __device__ __forceinline__ void ld_cols(float (&f)[4][HD / 16], const float* base, int64_t ld, int r0, int last, int c, int g) {
  constexpr int NT = HD / 16;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float* p = base + (int64_t)min(r0 + 4 * g + j, last) * ld + NT * c;
#pragma unroll
    for (int v = 0; v < NT / 4; ++v) {
      const f32x4 t = *reinterpret_cast<const f32x4*>(p + 4 * v);
#pragma unroll
      for (int e = 0; e < 4; ++e) f[j][4 * v + e] = t[e];
    }
  }
}
// acc[i][e] = D[column block i, row 4 g + e][c]: as float4 pieces of one row, piece q = e * (NT / 4) + v covers columns
// NT * (4 g + e) + 4 v ..
template <int HD> __device__ __forceinline__ f32x4 piece(const f32x4 (&acc)[HD / 16], int q) {
  constexpr int NT = HD / 16;
  const int e = q / (NT / 4), v = q % (NT / 4);
  return f32x4{acc[4 * v][e], acc[4 * v + 1][e], acc[4 * v + 2][e], acc[4 * v + 3][e]};
}
template <int HD> __device__ __forceinline__ int piece_col(int q, int g) {
  constexpr int NT = HD / 16;
  return NT * (4 * g + q / (NT / 4)) + 4 * (q % (NT / 4));
}
// A block of rows that some columns see and others do not (keys behind a query, rows past the end) is multiplied with weights that
// are zero for the pairs that do not count, which is right as long as the rows are finite: zero times an infinity or NaN is
// NaN.  `mul_seen`: acc += f^T . w with row 4 g + j counted only for the columns with ok[j], one row at a time, each column dropping
// the products of rows that it does not see.  It is far from the loops over the blocks, which carry no branch for it (a
// branch there costs the backward 4 %): the forward asks its last block, the only one with such pairs, whether its rows
// are finite (`odd_rows`) and leaves it for the end if they are not; the backward's wavefronts note on the way whether a score
// or delta, sums over whole rows, was not finite, and if so walk their blocks again.
template <int NT> __device__ __forceinline__ bool odd_rows(const float (&f)[4][NT]) {
  float t = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < NT; ++i) t = __builtin_fmaf(f[j][i], 0.f, t);            // 0, or NaN
  return __any(t != 0.f);
}
template <int NT> __device__ __forceinline__ void mul_seen(f32x4 (&acc)[NT], const float (&f)[4][NT], const f32x4& w, const bool (&ok)[4], int c, int g) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll 1
    for (int gg = 0; gg < 4; ++gg) {
      const bool see = __shfl((int)ok[j], 16 * gg + c, 64) != 0;
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const f32x4 p = mfma4(g == gg ? f[j][i] : 0.f, g == gg ? w[j] : 0.f, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][e] += see ? p[e] : 0.f;
        __builtin_amdgcn_sched_barrier(0);                       // one product at a time: no registers beyond the plain path's
      }
    }
}
__device__ __forceinline__ float max_g(float v) { v = fmaxf(v, __shfl_xor(v, 16, 64)); return fmaxf(v, __shfl_xor(v, 32, 64)); }
__device__ __forceinline__ float sum_g(float v) { v += __shfl_xor(v, 16, 64); return v + __shfl_xor(v, 32, 64); }

template <int HD>
__global__ __launch_bounds__(AW * 64) void attn32_fwd_kernel(AttnArgs a) {
  constexpr int NT = HD / 16;
  __shared__ f32x4 red[AW * NT * 64];
  __shared__ float red_m[AW][16], red_l[AW][16];
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * 16, head = blockIdx.y, ib = blockIdx.z;      // long rows first
  const int d = a.h * HD, dkv = a.hkv * HD, kvh = head / (a.h / a.hkv);
  const float* base = (const float*)a.qkv + (int64_t)ib * a.s * a.ld;
  const float *kp = base + d + kvh * HD, *vp = kp + dkv;
  const float scale = rsqrtf((float)HD);
  const int q = q0 + c, last = a.s - 1;
  f32x4 qf[NT];
  ld_rows<HD>(qf, base + (int64_t)min(q, last) * a.ld + head * HD, g);
  const int nblk = ((a.causal ? min(a.s, q0 + 16) : a.s) + 15) / 16;
  f32x4 o[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  f32x4 kf[NT];
  ld_rows<HD>(kf, kp + (int64_t)min(w * 16 + c, last) * a.ld, g);
  bool odd = false;                                      // the last block, the only one with keys a query does not see, waits for the end
  f32x4 sc;
  for (int kb = w; kb < nblk; kb += AW) {
    float vf[4][NT];
    ld_cols<HD>(vf, vp, a.ld, kb * 16, last, c, g);
    sc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) sc = mfma4(kf[t][j], qf[t][j], sc);
    ld_rows<HD>(kf, kp + (int64_t)min((kb + AW) * 16 + c, last) * a.ld, g);      // next block, in flight during the rest
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int key = kb * 16 + 4 * g + e;
      const bool ok = key < a.s && (!a.causal || key <= q);
      sc[e] = ok ? sc[e] * scale : -INFINITY;
      mx = fmaxf(mx, sc[e]);
    }
    const float mn = fmaxf(m, max_g(mx));
    const float sub = mn == -INFINITY ? 0.f : mn;                                 // nothing seen yet: exp(-inf) = 0
    const float alpha = expf(m - sub);
    float ps = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) { sc[e] = expf(sc[e] - sub); ps += sc[e]; }
    m = mn;
    l = l * alpha + ps;
#pragma unroll
    for (int i = 0; i < NT; ++i) o[i] *= alpha;
    if (kb == nblk - 1 && (odd = odd_rows(vf))) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < NT; ++i) vf[j][i] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < NT; ++i) o[i] = mfma4(vf[j][i], sc[j], o[i]);
  }
  if (odd) {
    float vf[4][NT];
    bool ok[4];
    ld_cols<HD>(vf, vp, a.ld, (nblk - 1) * 16, last, c, g);
#pragma unroll
    for (int e = 0; e < 4; ++e) { const int key = (nblk - 1) * 16 + 4 * g + e; ok[e] = key < a.s && (!a.causal || key <= q); }
    mul_seen(o, vf, sc, ok, c, g);
  }
  l = sum_g(l);
  if (g == 0) { red_m[w][c] = m; red_l[w][c] = l; }
#pragma unroll
  for (int p = 0; p < NT; ++p) red[(w * NT + p) * 64 + lane] = piece<HD>(o, p);
  __syncthreads();
  float mt = red_m[0][c];
#pragma unroll
  for (int k = 1; k < AW; ++k) mt = fmaxf(mt, red_m[k][c]);
  float f[AW], lt = 0.f;
#pragma unroll
  for (int k = 0; k < AW; ++k) { f[k] = red_m[k][c] == -INFINITY ? 0.f : expf(red_m[k][c] - mt); lt += red_l[k][c] * f[k]; }
  const float inv = 1.f / lt;
  if (q >= a.s) return;
#pragma unroll
  for (int t = 0; t < (NT + AW - 1) / AW; ++t) {
    const int p = w + t * AW;
    if (p >= NT) break;
    f32x4 v = red[p * 64 + lane] * f[0];
#pragma unroll
    for (int k = 1; k < AW; ++k) v += red[(k * NT + p) * 64 + lane] * f[k];
    *reinterpret_cast<f32x4*>((float*)a.o + ((int64_t)ib * a.s + q) * d + head * HD + piece_col<HD>(p, g)) = v * inv;
  }
  if (w == 0 && g == 0) a.lse[((int64_t)ib * a.h + head) * a.s + q] = mt == -INFINITY ? NAN : mt + logf(lt);
}

// dQ of the 16 queries from q0 on; leaves delta = rowsum(dO * O) as well
template <int HD>
__device__ __forceinline__ void attn32_dq(const AttnArgs& a, int q0, int head, int ib, f32x4* red) {
  constexpr int NT = HD / 16;
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int d = a.h * HD, dkv = a.hkv * HD, kvh = head / (a.h / a.hkv);
  const float* base = (const float*)a.qkv + (int64_t)ib * a.s * a.ld;
  const float *kp = base + d + kvh * HD, *vp = kp + dkv;
  const float scale = rsqrtf((float)HD);
  const int q = q0 + c, last = a.s - 1, qc = min(q, last);
  f32x4 qf[NT], dof[NT];
  ld_rows<HD>(qf, base + (int64_t)qc * a.ld + head * HD, g);
  ld_rows<HD>(dof, (const float*)a.dout + ((int64_t)ib * a.s + qc) * d + head * HD, g);
  float delta = 0.f;
  {
    f32x4 of[NT];
    ld_rows<HD>(of, (const float*)a.o + ((int64_t)ib * a.s + qc) * d + head * HD, g);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) delta += of[t][e] * dof[t][e];
    delta = sum_g(delta);
  }
  const int64_t si = ((int64_t)ib * a.h + head) * a.s + qc;
  if (w == 0 && g == 0 && q < a.s) a.delta[si] = delta;
  const float lse = a.lse[si];
  const int nblk = ((a.causal ? min(a.s, q0 + 16) : a.s) + 15) / 16;
  f32x4 dq[NT];
  float odd = 0.f;                                       // becomes NaN with the scores of a key row that holds an infinity or NaN
  auto walk = [&](auto seen_c) __attribute__((always_inline)) {
    constexpr bool seen = decltype(seen_c)::value;
#pragma unroll
    for (int i = 0; i < NT; ++i) dq[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kb = w; kb < nblk; kb += AW) {
      const int64_t kr = (int64_t)min(kb * 16 + c, last) * a.ld;
      f32x4 kf[NT], vf[NT];
      float kc[4][NT];
      ld_rows<HD>(kf, kp + kr, g);
      ld_rows<HD>(vf, vp + kr, g);
      ld_cols<HD>(kc, kp, a.ld, kb * 16, last, c, g);
      f32x4 sc = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) { sc = mfma4(kf[t][j], qf[t][j], sc); dp = mfma4(vf[t][j], dof[t][j], dp); }
      bool ok[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int key = kb * 16 + 4 * g + e;
        ok[e] = key < a.s && (!a.causal || key <= q);
        if (!seen) odd = __builtin_fmaf(sc[e], 0.f, odd);
        sc[e] = ok[e] ? expf(sc[e] * scale - lse) * (dp[e] - delta) : 0.f;
      }
      if (seen) mul_seen(dq, kc, sc, ok, c, g);
      else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < NT; ++i) dq[i] = mfma4(kc[j][i], sc[j], dq[i]);
      }
    }
  };
  walk(std::false_type{});
  if (__any(odd != 0.f)) walk(std::true_type{});
#pragma unroll
  for (int p = 0; p < NT; ++p) red[(w * NT + p) * 64 + lane] = piece<HD>(dq, p);
  __syncthreads();
  if (q >= a.s) return;
#pragma unroll
  for (int t = 0; t < (NT + AW - 1) / AW; ++t) {
    const int p = w + t * AW;
    if (p >= NT) break;
    f32x4 v = red[p * 64 + lane];
#pragma unroll
    for (int k = 1; k < AW; ++k) v += red[(k * NT + p) * 64 + lane];
    *reinterpret_cast<f32x4*>((float*)a.dqkv + ((int64_t)ib * a.s + q) * a.ld + head * HD + piece_col<HD>(p, g)) = v * scale;
  }
}

// dK and dV of the 16 keys from k0 on: the wavefronts take the (query head of the group, block of 16 queries) pairs in turn.
// K and V fragments wait in LDS (`kv`) in the order they are used in (registers hold two operand fragments in either direction
// and both sums).  delta of a block's queries is formed here again from dO and O, so that dQ can run at the same time.
template <int HD>
__device__ __forceinline__ void attn32_dkv(const AttnArgs& a, int k0, int kvh, int ib, f32x4* red, f32x4* kv) {
  constexpr int NT = HD / 16;
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int d = a.h * HD, dkv = a.hkv * HD, grp = a.h / a.hkv;
  const float* base = (const float*)a.qkv + (int64_t)ib * a.s * a.ld;
  const float* dob = (const float*)a.dout + (int64_t)ib * a.s * d;
  const float scale = rsqrtf((float)HD);
  const int key = k0 + c, last = a.s - 1;
  if (w < 2) {
    f32x4 f[NT];
    ld_rows<HD>(f, base + (int64_t)min(key, last) * a.ld + d + w * dkv + kvh * HD, g);
#pragma unroll
    for (int t = 0; t < NT; ++t) kv[(w * NT + t) * 64 + lane] = f[t];
  }
  __syncthreads();
  f32x4 dk[NT], dv[NT];
  const int qb0 = a.causal ? k0 / 16 : 0, nqb = (a.s + 15) / 16 - qb0;
  float odd = 0.f;                                       // becomes NaN with the scores or delta of a row of Q or dO that holds an infinity or NaN
  auto walk = [&](auto seen_c) __attribute__((always_inline)) {
    constexpr bool seen = decltype(seen_c)::value;
#pragma unroll
    for (int i = 0; i < NT; ++i) dk[i] = dv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int it = w; it < grp * nqb; it += AW) {
      const int head = kvh * grp + it / nqb, q0 = (qb0 + it % nqb) * 16;
      const float *qh = base + head * HD, *doh = dob + head * HD;
      const int qr = min(q0 + c, last);
      f32x4 qf[NT], dof[NT];
      float qc[4][NT], doc[4][NT];
      ld_rows<HD>(qf, qh + (int64_t)qr * a.ld, g);
      ld_rows<HD>(dof, doh + (int64_t)qr * d, g);
      ld_cols<HD>(doc, doh, d, q0, last, c, g);
      if (!seen) ld_cols<HD>(qc, qh, a.ld, q0, last, c, g);
      const float* lse = a.lse + ((int64_t)ib * a.h + head) * a.s;
      float ls[4], dl[4], dc = 0.f;
      {
        f32x4 of[NT];
        ld_rows<HD>(of, (const float*)a.o + ((int64_t)ib * a.s + qr) * d + head * HD, g);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) dc += of[t][e] * dof[t][e];
        dc = sum_g(dc);                                    // delta of query q0 + c
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) { ls[e] = lse[min(q0 + 4 * g + e, last)]; dl[e] = __shfl(dc, 4 * g + e, 64); }
      f32x4 sc = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const f32x4 kf = kv[t * 64 + lane], vf = kv[(NT + t) * 64 + lane];
#pragma unroll
        for (int j = 0; j < 4; ++j) { sc = mfma4(qf[t][j], kf[j], sc); dp = mfma4(dof[t][j], vf[j], dp); }
      }
      bool ok[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int q = q0 + 4 * g + e;
        ok[e] = q < a.s && (!a.causal || key <= q);
        if (!seen) odd = __builtin_fmaf(sc[e], 0.f, odd);
        const float p = ok[e] ? expf(sc[e] * scale - ls[e]) : 0.f;
        sc[e] = p;
        dp[e] = ok[e] ? p * (dp[e] - dl[e]) : 0.f;
      }
      if (seen) {
        mul_seen(dv, doc, sc, ok, c, g);
        ld_cols<HD>(qc, qh, a.ld, q0, last, c, g);          // (both at once do not fit the registers)
        mul_seen(dk, qc, dp, ok, c, g);
      } else {
        odd = __builtin_fmaf(dc, 0.f, odd);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < NT; ++i) {
            dv[i] = mfma4(doc[j][i], sc[j], dv[i]);
            dk[i] = mfma4(qc[j][i], dp[j], dk[i]);
          }
      }
    }
  };
  walk(std::false_type{});
  if (__any(odd != 0.f)) walk(std::true_type{});
  // the wavefronts' sums, dK first, then dV
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    if (which) __syncthreads();
#pragma unroll
    for (int p = 0; p < NT; ++p) red[(w * NT + p) * 64 + lane] = which ? piece<HD>(dv, p) : piece<HD>(dk, p);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < (NT + AW - 1) / AW; ++t) {
      const int p = w + t * AW;
      if (p >= NT || key >= a.s) break;
      f32x4 v = red[p * 64 + lane];
#pragma unroll
      for (int k = 1; k < AW; ++k) v += red[(k * NT + p) * 64 + lane];
      *reinterpret_cast<f32x4*>((float*)a.dqkv + ((int64_t)ib * a.s + key) * a.ld + d + which * dkv + kvh * HD + piece_col<HD>(p, g)) = which ? v : v * scale;
    }
  }
}

// Both halves of the backward in one launch: a grid of dK/dV workgroups (low keys first: they see the most queries), then
// one of dQ workgroups (late queries first).  Neither half alone fills the chip at the lengths fp32 stages have: two launches
// took 48 us, one takes 28 (448 positions, 4 heads of 128); 155 and 126 us at 2 x 700, 8 heads of 128.
template <int HD>
__global__ __launch_bounds__(AW * 64) void attn32_bwd_kernel(AttnArgs a) {
  __shared__ f32x4 red[AW * (HD / 16) * 64], kv[2 * (HD / 16) * 64];
  const int nb = (a.s + 15) / 16, n_kv = nb * a.hkv * a.b;
  int id = blockIdx.x;
  if (id < n_kv) {
    const int blk = id / (a.hkv * a.b), r = id % (a.hkv * a.b);
    attn32_dkv<HD>(a, blk * 16, r % a.hkv, r / a.hkv, red, kv);
  } else {
    id -= n_kv;
    const int blk = id / (a.h * a.b), r = id % (a.h * a.b);
    attn32_dq<HD>(a, (nb - 1 - blk) * 16, r % a.h, r / a.h, red);
  }
}

}  // namespace

bool attn32_supported(const AttnArgs& a) {
  auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  return (a.hd == 64 || a.hd == 128) && a.s >= 1 && a.ld % 4 == 0 && al16(a.qkv) && al16(a.o) && al16(a.dout) && al16(a.dqkv) &&
         a.b <= 65535 && a.h <= 65535 && (int64_t)((a.s + 15) / 16) * (a.h + a.hkv) * a.b < (1 << 23);
}

hipError_t attn32_fwd(const AttnArgs& a, hipStream_t s) {
  const dim3 grid((a.s + 15) / 16, a.h, a.b);
  if (a.hd == 64) hipLaunchKernelGGL((attn32_fwd_kernel<64>), grid, dim3(AW * 64), 0, s, a);
  else hipLaunchKernelGGL((attn32_fwd_kernel<128>), grid, dim3(AW * 64), 0, s, a);
  return hipGetLastError();
}

hipError_t attn32_bwd(const AttnArgs& a, hipStream_t s) {
  const int64_t grid = (int64_t)((a.s + 15) / 16) * (a.hkv + a.h) * a.b;
  if (a.hd == 64) hipLaunchKernelGGL((attn32_bwd_kernel<64>), dim3((unsigned)grid), dim3(AW * 64), 0, s, a);
  else hipLaunchKernelGGL((attn32_bwd_kernel<128>), dim3((unsigned)grid), dim3(AW * 64), 0, s, a);
  return hipGetLastError();
}

}  // namespace stg
