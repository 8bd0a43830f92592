// FP64 MFMA kernels of the blocked Gram-Schmidt: the split-K projection
// product (R_bar = Qbar^T Q_t, S = Q_prev^T P, Gram matrices), the rank-K
// update (Q_t -= Qbar R_bar, P -= Q_prev S), the panel's Cholesky step and the
// in-place triangular transform of the panel (P <- P R^{-1}).
//
// MFMA layout used throughout (v_mfma_f64_16x16x4, one wavefront of 64 lanes):
// D = X Y + D with X 16x4, Y 4x16; lane l supplies X[l%16][l/16] and
// Y[l/16][l%16] and holds D[4r + l/16][l%16] in accumulator element r.  Every
// product is issued as the transposed product (D = C^T), so lane l holds
// C[i0 + l%16][j0 + 4r + l/16]: sixteen consecutive rows of a column-major C
// per lane group, i.e. whole 128-byte lines on load and store.  Within a group
// of 16 k-values lane l contributes k = k0 + 4*(l/16) + s in MFMA step s (one
// fixed permutation of the reduction index, shared by both operands).
//
// Reductions over long K are split across blocks; partial tiles go to the
// workspace and a second small kernel sums them in split order, so results do
// not depend on scheduling and no device-wide fence is needed.
#include "cqr_colwise.hpp"
#include "cqr_kernels.hpp"
#include "cqr_mfma.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace cqr {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

// FP32 product of FP64 operands rounded to FP32 (the mixed-precision
// coefficient product R_bar = Qbar^T Q_t).  Operand lanes as in the FP64 form.
// The product kernels accumulate it in FP32 over 16 k-values only (four MFMA
// steps) and add each group's sums into FP64 accumulators, so the rounding of
// the reduction does not grow with K.
__device__ __forceinline__ v4f mfma(double x, double y, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32((float)x, (float)y, c, 0, 0, 0);
}

__device__ __forceinline__ v4f mfma(float x, float y, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0);
}

// Operand type of the product kernels' MFMA steps.
template <bool F32> struct OpT { typedef double type; };
template <> struct OpT<true> { typedef float type; };

// acc += t, element by element in FP64 (one slab's FP32 sums into the FP64
// accumulators of the mixed-precision product).
__device__ __forceinline__ void widen_add(v4d& acc, const v4f& t) {
#pragma unroll
  for (int r = 0; r < 4; ++r) acc[r] += (double)t[r];
}

// Result layout of the transposed-issue 16x16x4 products: lane (li, g),
// register r holds C[i0 + li][j0 + colsub(r, g)] -- the FP64 form spreads a
// lane's four values over columns g, g+4, g+8, g+12, the FP32 form over the
// consecutive columns 4g .. 4g+3.
__device__ __forceinline__ int colsub(int r, int g, bool f32) { return f32 ? 4 * g + r : 4 * r + g; }


// Partial-tile layout shared by the product and reduction kernels: tile
// `tile` of split `sp`, wave w, accumulator element q (16 per lane), lane l at
// part[((sp * ntiles + tile) * 4 + w) * 1024 + q * 64 + l].
__device__ __forceinline__ int64_t part_off(int sp, int ntiles, int tile, int wave) {
  return (((int64_t)sp * ntiles + tile) * 4 + wave) * 1024;
}

// Sum over splits of four element slots q = 4 qg + u (u < 4) of one wave's
// partial tiles, lane `lane`, in split order.  Batches of kB splits have all
// their loads issued before the first addition.
template <int kB = 16>
__device__ __forceinline__ void sum_partials4(const double* part, int nsplit, int ntiles, int tile, int wave,
                                              int qg, int lane, double (&v)[4]) {
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = 0.0;
  const double* base = part + part_off(0, ntiles, tile, wave) + 4 * qg * 64 + lane;
  const int64_t sstride = (int64_t)ntiles * 4 * 1024;
  for (int sp0 = 0; sp0 < nsplit; sp0 += kB) {
    double t[kB][4];
#pragma unroll
    for (int k = 0; k < kB; ++k) {
      const int sp = std::min(sp0 + k, nsplit - 1);       // clamped: extra loads are discarded
#pragma unroll
      for (int u = 0; u < 4; ++u) t[k][u] = base[sp * sstride + u * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kB; ++k)
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] += (sp0 + k < nsplit) ? t[k][u] : 0.0;
  }
}

// --------------------------------------------------------------------------
// Split-K product  C = A^T B  (A: K x M, B: K x N, both K-contiguous).
// Tile 64x64 per block, 4 waves each a 32x32 quadrant.  Operand slabs of
// KC = 32 k-values are staged through LDS (double-buffered): each global load
// instruction covers 4 columns x 256 contiguous bytes.  Requires 16-byte
// aligned operands with even leading dimensions (else tn_direct_kernel).
// --------------------------------------------------------------------------

constexpr int KC = 32;           // k-values per LDS slab
constexpr int LDP = KC + 2;      // padded LDS column (doubles)

// Store a wave's 32 x 32 quadrant (16 values per lane, element (x, y, r) at
// row i0 + 16x + li, column j0 + 16y + 4r + g) to C, and add it into C2 if
// given; the C2 loads are all issued before any store.
__device__ __forceinline__ void store_quadrant(double* C, int64_t ldc, double* C2, int64_t ldc2, int M, int M2,
                                               int N, int i0, int j0, int li, int g, bool f32,
                                               const double (&v)[16]) {
  double old[16];
  if (C2) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int x = e >> 3, y = (e >> 2) & 1, r = e & 3;
      const int i = i0 + 16 * x + li, j = j0 + 16 * y + colsub(r, g, f32);
      old[e] = (i < M2 && j < N) ? C2[i + (int64_t)j * ldc2] : 0.0;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int x = e >> 3, y = (e >> 2) & 1, r = e & 3;
    const int i = i0 + 16 * x + li, j = j0 + 16 * y + colsub(r, g, f32);
    if (i < M && j < N) {
      if (C) C[i + (int64_t)j * ldc] = v[e];
      if (C2 && i < M2) C2[i + (int64_t)j * ldc2] = old[e] + v[e];
    }
  }
}

template <class Acc>
__device__ __forceinline__ void tn_store(const TnArgs& a, const Acc (&acc)[2][2], int tile, int split, int wave,
                                         int lane, int i0, int j0, bool f32_layout) {
  const int li = lane & 15, g = lane >> 4;
  if (a.nsplit > 1) {
    double* mine = a.part + part_off(split, a.ntiles, tile, wave);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[((x * 2 + y) * 4 + r) * 64 + lane] = acc[x][y][r];
    return;
  }
  double v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = acc[e >> 3][(e >> 2) & 1][e & 3];
  store_quadrant(a.C, a.ldc, a.C2, a.ldc2, a.M, a.M2, a.N, i0, j0, li, g, f32_layout, v);
}

template <int TAG, bool F32>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void tn_lds_kernel(TnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  typedef v4d Acc;    // FP64 accumulators (FP32 products are widened per slab)
  typedef typename OpT<F32>::type Op;
  __shared__ double sA[2][64 * LDP];
  __shared__ double sB[2][64 * LDP];
  const int tile = blockIdx.x, split = blockIdx.y;
  const int tm = tile / a.tilesN, tn = tile % a.tilesN;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int64_t kb = (int64_t)split * a.kchunk;
  const int64_t ke = std::min<int64_t>(a.K, kb + a.kchunk);
  // staging: thread loads one v2d (k pair lq) of columns lc + 16r, r < 4
  const int lc = tid >> 4, lq = tid & 15;
  const double* ga[4];
  const double* gb[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    int ia = tm * 64 + lc + 16 * r, jb = tn * 64 + lc + 16 * r;
    // columns outside the matrix read column 0 and feed only unstored outputs
    ga[r] = a.A + (int64_t)(ia < a.M ? ia : 0) * a.lda + 2 * lq;
    gb[r] = a.B + (int64_t)(jb < a.N ? jb : 0) * a.ldb + 2 * lq;
  }
  Acc acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = Acc{0, 0, 0, 0};
  const int ia0 = (wave & 1) * 32, jb0 = (wave >> 1) * 32;
  const int nfull = (int)((ke - kb) / KC);

  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < KC; kk += 16) {
      [[maybe_unused]] v4f t32[2][2];
      if constexpr (F32)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) t32[x][y] = v4f{0, 0, 0, 0};
      Op xa[2][4], xb[2][4];   // FP32 operands are rounded as they leave LDS
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const double* pa = &sA[buf][(ia0 + 16 * t + li) * LDP + kk + 4 * g];
        const double* pb = &sB[buf][(jb0 + 16 * t + li) * LDP + kk + 4 * g];
        v2d a0 = *reinterpret_cast<const v2d*>(pa), a1 = *reinterpret_cast<const v2d*>(pa + 2);
        v2d b0 = *reinterpret_cast<const v2d*>(pb), b1 = *reinterpret_cast<const v2d*>(pb + 2);
        xa[t][0] = a0.x; xa[t][1] = a0.y; xa[t][2] = a1.x; xa[t][3] = a1.y;
        xb[t][0] = b0.x; xb[t][1] = b0.y; xb[t][2] = b1.x; xb[t][3] = b1.y;
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) {
            if constexpr (F32)
              t32[x][y] = mfma(xb[y][s], xa[x][s], t32[x][y]);
            else
              acc[x][y] = mfma(xb[y][s], xa[x][s], acc[x][y]);
          }
      if constexpr (F32)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) widen_add(acc[x][y], t32[x][y]);
    }
  };
  // slab sl's first k (clamped to the last full slab: prefetches past the end
  // reload cached data that is never used)
  auto koff = [&](int sl) { return kb + (int64_t)std::min(sl, nfull - 1) * KC; };

  if (nfull > 0) {
    // three-stage pipeline: slab sl in LDS is multiplied while the register
    // set of slab sl+1 (issued one slab earlier) lands and slab sl+2 is
    // requested into the other set; the two sets alternate explicitly
    v2d ra0[4], rb0[4], ra1[4], rb1[4];
#define CQR_TN_LOAD(RA, RB, K) {                                        \
    RA[0] = *reinterpret_cast<const v2d*>(ga[0] + (K));              \
    RB[0] = *reinterpret_cast<const v2d*>(gb[0] + (K));              \
    RA[1] = *reinterpret_cast<const v2d*>(ga[1] + (K));              \
    RB[1] = *reinterpret_cast<const v2d*>(gb[1] + (K));              \
    RA[2] = *reinterpret_cast<const v2d*>(ga[2] + (K));              \
    RB[2] = *reinterpret_cast<const v2d*>(gb[2] + (K));              \
    RA[3] = *reinterpret_cast<const v2d*>(ga[3] + (K));              \
    RB[3] = *reinterpret_cast<const v2d*>(gb[3] + (K));              \
  }
#define CQR_TN_PUT(BUF, RA, RB) {                                       \
    *reinterpret_cast<v2d*>(&sA[BUF][(lc + 0) * LDP + 2 * lq]) = RA[0];      \
    *reinterpret_cast<v2d*>(&sB[BUF][(lc + 0) * LDP + 2 * lq]) = RB[0];      \
    *reinterpret_cast<v2d*>(&sA[BUF][(lc + 16) * LDP + 2 * lq]) = RA[1];      \
    *reinterpret_cast<v2d*>(&sB[BUF][(lc + 16) * LDP + 2 * lq]) = RB[1];      \
    *reinterpret_cast<v2d*>(&sA[BUF][(lc + 32) * LDP + 2 * lq]) = RA[2];      \
    *reinterpret_cast<v2d*>(&sB[BUF][(lc + 32) * LDP + 2 * lq]) = RB[2];      \
    *reinterpret_cast<v2d*>(&sA[BUF][(lc + 48) * LDP + 2 * lq]) = RA[3];      \
    *reinterpret_cast<v2d*>(&sB[BUF][(lc + 48) * LDP + 2 * lq]) = RB[3];      \
  }
    CQR_TN_LOAD(ra0, rb0, koff(0))
    CQR_TN_LOAD(ra1, rb1, koff(1))
    CQR_TN_PUT(0, ra0, rb0)
    __syncthreads();
    int sl = 0;
    for (; sl + 2 <= nfull; sl += 2) {
      CQR_TN_LOAD(ra0, rb0, koff(sl + 2))
      __builtin_amdgcn_sched_barrier(0);
      compute(0);
      __builtin_amdgcn_sched_barrier(0);
      CQR_TN_PUT(1, ra1, rb1)
      __syncthreads();
      CQR_TN_LOAD(ra1, rb1, koff(sl + 3))
      __builtin_amdgcn_sched_barrier(0);
      compute(1);
      __builtin_amdgcn_sched_barrier(0);
      CQR_TN_PUT(0, ra0, rb0)
      __syncthreads();
    }
    if (sl < nfull) compute(0);
#undef CQR_TN_LOAD
#undef CQR_TN_PUT
  }
  const int64_t kt = kb + (int64_t)nfull * KC;
  if (kt < ke) {
    // partial last slab: masked scalar loads, zero beyond ke
    const int buf = nfull & 1;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t k = kt + 2 * lq;
      const double* pa = ga[r] - 2 * lq;
      const double* pb = gb[r] - 2 * lq;
      v2d va, vb;
      va.x = (k < ke) ? pa[k] : 0.0;
      va.y = (k + 1 < ke) ? pa[k + 1] : 0.0;
      vb.x = (k < ke) ? pb[k] : 0.0;
      vb.y = (k + 1 < ke) ? pb[k + 1] : 0.0;
      *reinterpret_cast<v2d*>(&sA[buf][(lc + 16 * r) * LDP + 2 * lq]) = va;
      *reinterpret_cast<v2d*>(&sB[buf][(lc + 16 * r) * LDP + 2 * lq]) = vb;
    }
    __syncthreads();
    compute(buf);
  }
  tn_store(a, acc, tile, split, wave, lane, tm * 64 + ia0, tn * 64 + jb0, F32);
}

// The same product with 16-deep slabs (36 KB of LDS, three waves per SIMD),
// taken by FP32 products with at least two tile rows and two or three tile
// columns whose depth is not a multiple of 32 (tnf_kernel takes the others;
// with four or more tile columns, such products take tn2_kernel).  An FP32 MFMA
// takes fewer cycles than the FP64 one, so the FP32 product waits more on its
// loads and the third wave hides them (the n = 16384 factorization with FP32
// updates runs 5% faster); in FP64 the twice as many barriers of the shorter
// slabs cost more than the extra wave returns (about 1% slower at n = 16384
// and n = 32768), and FP64 products keep tn_lds_kernel.
// Thread (lc, lq) stages one v2d (k pair lq) of columns lc + 32 q, q < 2, of
// each operand per slab; the pipeline, the tile order and the output contract
// (partials or C, C2) are those of tn_lds_kernel.
template <int TAG, bool F32>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void tn16_kernel(TnArgs a) {
  constexpr int SK = 16, LW = SK + 2, NQ = 2, TPC = SK / 2, CPP = 256 / TPC;
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  typedef v4d Acc;    // FP64 accumulators (FP32 products are widened per slab)
  typedef typename OpT<F32>::type Op;
  __shared__ double sA[2][64 * LW];
  __shared__ double sB[2][64 * LW];
  const int tile = blockIdx.x, split = blockIdx.y;
  const int tm = tile / a.tilesN, tn = tile % a.tilesN;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int64_t kb = (int64_t)split * a.kchunk;
  const int64_t ke = std::min<int64_t>(a.K, kb + a.kchunk);
  const int lc = tid / TPC, lq = tid % TPC;
  const double* ga[NQ];
  const double* gb[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int ia = tm * 64 + lc + CPP * q, jb = tn * 64 + lc + CPP * q;
    // columns outside the matrix read column 0 and feed only unstored outputs
    ga[q] = a.A + (int64_t)(ia < a.M ? ia : 0) * a.lda + 2 * lq;
    gb[q] = a.B + (int64_t)(jb < a.N ? jb : 0) * a.ldb + 2 * lq;
  }
  Acc acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = Acc{0, 0, 0, 0};
  const int ia0 = (wave & 1) * 32, jb0 = (wave >> 1) * 32;
  const int nfull = (int)((ke - kb) / SK);
  auto compute = [&](int buf) {
    Op xa[2][4], xb[2][4];   // FP32 operands are rounded as they leave LDS
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const double* pa = &sA[buf][(ia0 + 16 * t + li) * LW + 4 * g];
      const double* pb = &sB[buf][(jb0 + 16 * t + li) * LW + 4 * g];
      v2d a0 = *reinterpret_cast<const v2d*>(pa), a1 = *reinterpret_cast<const v2d*>(pa + 2);
      v2d b0 = *reinterpret_cast<const v2d*>(pb), b1 = *reinterpret_cast<const v2d*>(pb + 2);
      xa[t][0] = a0.x; xa[t][1] = a0.y; xa[t][2] = a1.x; xa[t][3] = a1.y;
      xb[t][0] = b0.x; xb[t][1] = b0.y; xb[t][2] = b1.x; xb[t][3] = b1.y;
    }
    [[maybe_unused]] v4f t32[2][2];
    if constexpr (F32)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) t32[x][y] = v4f{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          if constexpr (F32)
            t32[x][y] = mfma(xb[y][s], xa[x][s], t32[x][y]);
          else
            acc[x][y] = mfma(xb[y][s], xa[x][s], acc[x][y]);
        }
    if constexpr (F32)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) widen_add(acc[x][y], t32[x][y]);
  };
  auto koff = [&](int sl) { return kb + (int64_t)std::min(sl, nfull - 1) * SK; };
  v2d ra0[NQ], rb0[NQ], ra1[NQ], rb1[NQ];
  auto load = [&](v2d (&ra)[NQ], v2d (&rb)[NQ], int64_t k) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      ra[q] = *reinterpret_cast<const v2d*>(ga[q] + k);
      rb[q] = *reinterpret_cast<const v2d*>(gb[q] + k);
    }
  };
  auto put = [&](int buf, const v2d (&ra)[NQ], const v2d (&rb)[NQ]) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      *reinterpret_cast<v2d*>(&sA[buf][(lc + CPP * q) * LW + 2 * lq]) = ra[q];
      *reinterpret_cast<v2d*>(&sB[buf][(lc + CPP * q) * LW + 2 * lq]) = rb[q];
    }
  };
  if (nfull > 0) {
    load(ra0, rb0, koff(0));
    load(ra1, rb1, koff(1));
    put(0, ra0, rb0);
    __syncthreads();
    int sl = 0;
    for (; sl + 2 <= nfull; sl += 2) {
      load(ra0, rb0, koff(sl + 2));
      __builtin_amdgcn_sched_barrier(0);
      compute(0);
      __builtin_amdgcn_sched_barrier(0);
      put(1, ra1, rb1);
      __syncthreads();
      load(ra1, rb1, koff(sl + 3));
      __builtin_amdgcn_sched_barrier(0);
      compute(1);
      __builtin_amdgcn_sched_barrier(0);
      put(0, ra0, rb0);
      __syncthreads();
    }
    if (sl < nfull) compute(0);
  }
  const int64_t kt = kb + (int64_t)nfull * SK;
  if (kt < ke) {
    // partial last slab: masked scalar loads, zero beyond ke
    const int buf = nfull & 1;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int64_t k = kt + 2 * lq;
      const double* pa = ga[q] - 2 * lq;
      const double* pb = gb[q] - 2 * lq;
      v2d va, vb;
      va.x = (k < ke) ? pa[k] : 0.0;
      va.y = (k + 1 < ke) ? pa[k + 1] : 0.0;
      vb.x = (k < ke) ? pb[k] : 0.0;
      vb.y = (k + 1 < ke) ? pb[k + 1] : 0.0;
      *reinterpret_cast<v2d*>(&sA[buf][(lc + CPP * q) * LW + 2 * lq]) = va;
      *reinterpret_cast<v2d*>(&sB[buf][(lc + CPP * q) * LW + 2 * lq]) = vb;
    }
    __syncthreads();
    compute(buf);
  }
  tn_store(a, acc, tile, split, wave, lane, tm * 64 + ia0, tn * 64 + jb0, F32);
}

// Two tile rows per workgroup (512 threads): waves 0-3 compute tile row
// 2 tp, waves 4-7 tile row 2 tp + 1, both over the same staged slab of B, so
// B's columns are read once per pair of tile rows.  16-deep slabs (55 KB of
// LDS).  Thread (lc, lq) stages k pair lq of A's columns lc and lc + 64 and
// of B's column lc.  Each wave stores its 32 x 32 quadrant of its own 64 x 64
// tile with the contract of tn_lds_kernel (a missing second tile row of an
// odd tilesM stages and computes but stores nothing).
// Taken by the products with at least two tile rows and four tile columns
// that the 128 x 128 kernels do not take: FP32 ones whose depth is not a
// multiple of 32 (tnf_kernel) and FP64 ones whose depth is not a multiple of
// 16 (tnq_kernel).  Alone, the K = 49152, 256 x 32768 FP64 product
// ran at 63 TFLOP/s on it against 55 for tn_lds_kernel (tnq_kernel: 65-67).
template <int TAG, bool F32>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void tn2_kernel(TnArgs a) {
  constexpr int SK = 16, LW = SK + 2;
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  typedef v4d Acc;    // FP64 accumulators (FP32 products are widened per slab)
  typedef typename OpT<F32>::type Op;
  __shared__ double sA[2][128 * LW];
  __shared__ double sB[2][64 * LW];
  const int tp = blockIdx.x / a.tilesN, tn = blockIdx.x % a.tilesN, split = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int h = wave >> 2, w4 = wave & 3;
  const int tm = 2 * tp + h;
  const int64_t kb = (int64_t)split * a.kchunk;
  const int64_t ke = std::min<int64_t>(a.K, kb + a.kchunk);
  const int lc = tid >> 3, lq = tid & 7;
  const double* ga[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int ia = tp * 128 + lc + 64 * q;
    // columns outside the matrix read column 0 and feed only unstored outputs
    ga[q] = a.A + (int64_t)(ia < a.M ? ia : 0) * a.lda + 2 * lq;
  }
  const int jb = tn * 64 + lc;
  const double* gb = a.B + (int64_t)(jb < a.N ? jb : 0) * a.ldb + 2 * lq;
  Acc acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = Acc{0, 0, 0, 0};
  const int ia0 = h * 64 + (w4 & 1) * 32, jb0 = (w4 >> 1) * 32;
  const int nfull = (int)((ke - kb) / SK);
  auto compute = [&](int buf) {
    Op xa[2][4], xb[2][4];   // FP32 operands are rounded as they leave LDS
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const double* pa = &sA[buf][(ia0 + 16 * t + li) * LW + 4 * g];
      const double* pb = &sB[buf][(jb0 + 16 * t + li) * LW + 4 * g];
      v2d a0 = *reinterpret_cast<const v2d*>(pa), a1 = *reinterpret_cast<const v2d*>(pa + 2);
      v2d b0 = *reinterpret_cast<const v2d*>(pb), b1 = *reinterpret_cast<const v2d*>(pb + 2);
      xa[t][0] = a0.x; xa[t][1] = a0.y; xa[t][2] = a1.x; xa[t][3] = a1.y;
      xb[t][0] = b0.x; xb[t][1] = b0.y; xb[t][2] = b1.x; xb[t][3] = b1.y;
    }
    [[maybe_unused]] v4f t32[2][2];
    if constexpr (F32)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) t32[x][y] = v4f{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          if constexpr (F32)
            t32[x][y] = mfma(xb[y][s], xa[x][s], t32[x][y]);
          else
            acc[x][y] = mfma(xb[y][s], xa[x][s], acc[x][y]);
        }
    if constexpr (F32)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) widen_add(acc[x][y], t32[x][y]);
  };
  auto koff = [&](int sl) { return kb + (int64_t)std::min(sl, nfull - 1) * SK; };
  v2d ra0[2], rb0, ra1[2], rb1;
  auto load = [&](v2d (&ra)[2], v2d& rb, int64_t k) {
    ra[0] = *reinterpret_cast<const v2d*>(ga[0] + k);
    ra[1] = *reinterpret_cast<const v2d*>(ga[1] + k);
    rb = *reinterpret_cast<const v2d*>(gb + k);
  };
  auto put = [&](int buf, const v2d (&ra)[2], const v2d& rb) {
    *reinterpret_cast<v2d*>(&sA[buf][lc * LW + 2 * lq]) = ra[0];
    *reinterpret_cast<v2d*>(&sA[buf][(lc + 64) * LW + 2 * lq]) = ra[1];
    *reinterpret_cast<v2d*>(&sB[buf][lc * LW + 2 * lq]) = rb;
  };
  if (nfull > 0) {
    load(ra0, rb0, koff(0));
    load(ra1, rb1, koff(1));
    put(0, ra0, rb0);
    __syncthreads();
    int sl = 0;
    for (; sl + 2 <= nfull; sl += 2) {
      load(ra0, rb0, koff(sl + 2));
      __builtin_amdgcn_sched_barrier(0);
      compute(0);
      __builtin_amdgcn_sched_barrier(0);
      put(1, ra1, rb1);
      __syncthreads();
      load(ra1, rb1, koff(sl + 3));
      __builtin_amdgcn_sched_barrier(0);
      compute(1);
      __builtin_amdgcn_sched_barrier(0);
      put(0, ra0, rb0);
      __syncthreads();
    }
    if (sl < nfull) compute(0);
  }
  const int64_t kt = kb + (int64_t)nfull * SK;
  if (kt < ke) {
    // partial last slab: masked scalar loads, zero beyond ke
    const int buf = nfull & 1;
    const int64_t k = kt + 2 * lq;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double* p = (q < 2 ? ga[q] : gb) - 2 * lq;
      v2d v;
      v.x = (k < ke) ? p[k] : 0.0;
      v.y = (k + 1 < ke) ? p[k + 1] : 0.0;
      double* d = q < 2 ? &sA[buf][(lc + 64 * q) * LW + 2 * lq] : &sB[buf][lc * LW + 2 * lq];
      *reinterpret_cast<v2d*>(d) = v;
    }
    __syncthreads();
    compute(buf);
  }
  if (tm < a.ntiles / a.tilesN)
    tn_store(a, acc, tm * a.tilesN + tn, split, w4, lane, tm * 64 + (w4 & 1) * 32, tn * 64 + jb0, F32);
}

// 128 x 128 output per workgroup (512 threads, 2 x 4 waves, each wave 64
// rows x 32 columns: a 4 x 2 grid of 16 x 16 MFMA blocks), FP64, 16-deep
// slabs (72 KB of LDS) with one register set of staged loads (slab s + 1 is
// requested while slab s is multiplied), two workgroups per CU.  K a
// multiple of 16 (a masked last slab would not fit the 128 registers).  Each
// operand column staged is reused by 128 output columns (tn2_kernel: 64 or
// 128), which halves the L2 requests per flop.  Alone, the K = 49152
// products with 256 rows run at 67 TFLOP/s against 62 for tn2_kernel (the
// clock under FP64 MFMA load is ~2.2 GHz, not 2.4, and the MFMA pipes are
// busy ~80% of those cycles).  The output contract is tn_lds_kernel's on the
// 64 x 64 tiles the workgroup covers: wave (wi, wj) holds rows 64 wi .. +64
// and columns 32 wj .. +32, i.e. quadrants (0, wj % 2) and (1, wj % 2) of
// tile (2 tp + wi, 2 tq + wj / 2).  Tiles are taken with the row index
// fastest, so the workgroups that read the same columns of B are adjacent.
template <int TAG>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void tnq_kernel(TnArgs a) {
  constexpr int SK = 16, LW = SK + 2, TPC = SK / 2, CPP = 512 / TPC;   // 8 threads per column, 64 columns a pass
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ double sA[2][128 * LW];
  __shared__ double sB[2][128 * LW];
  const int tilesM = a.ntiles / a.tilesN;
  const int qm = (tilesM + 1) / 2;
  int tp = blockIdx.x % qm, tq = blockIdx.x / qm;
  const int split = blockIdx.y;
  if (a.lower) {                       // blocks on and below the diagonal, row by row
    tp = (int)((sqrtf(8.0f * blockIdx.x + 1.0f) - 1.0f) * 0.5f);
    if (tp * (tp + 1) / 2 > (int)blockIdx.x) --tp;
    if ((tp + 1) * (tp + 2) / 2 <= (int)blockIdx.x) ++tp;
    tq = blockIdx.x - tp * (tp + 1) / 2;
  }
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int wi = wave & 1, wj = wave >> 1;
  const int ia0 = 64 * wi, jb0 = 32 * wj;
  const int64_t kb = (int64_t)split * a.kchunk;
  const int64_t ke = std::min<int64_t>(a.K, kb + a.kchunk);
  const int lc = tid / TPC, lq = tid % TPC;
  const double* ga[2];
  const double* gb[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int i = tp * 128 + lc + CPP * q, j = tq * 128 + lc + CPP * q;
    // columns outside the matrix read column 0 and feed only unstored outputs
    ga[q] = a.A + (int64_t)(i < a.M ? i : 0) * a.lda + 2 * lq;
    gb[q] = a.B + (int64_t)(j < a.N ? j : 0) * a.ldb + 2 * lq;
  }
  v4d acc[4][2];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = v4d{0, 0, 0, 0};
  auto compute = [&](int buf) {
#pragma unroll
    for (int s0 = 0; s0 < 4; s0 += 2) {
      double xa[4][2], xb[2][2];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const v2d v = *reinterpret_cast<const v2d*>(&sA[buf][(ia0 + 16 * t + li) * LW + 4 * g + s0]);
        xa[t][0] = v.x; xa[t][1] = v.y;
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const v2d v = *reinterpret_cast<const v2d*>(&sB[buf][(jb0 + 16 * t + li) * LW + 4 * g + s0]);
        xb[t][0] = v.x; xb[t][1] = v.y;
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) acc[x][y] = mfma(xb[y][s], xa[x][s], acc[x][y]);
    }
  };
  const int nfull = (int)((ke - kb) / SK);
  v2d ra[2], rb[2];
  auto load = [&](int64_t k) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      ra[q] = *reinterpret_cast<const v2d*>(ga[q] + k);
      rb[q] = *reinterpret_cast<const v2d*>(gb[q] + k);
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      *reinterpret_cast<v2d*>(&sA[buf][(lc + CPP * q) * LW + 2 * lq]) = ra[q];
      *reinterpret_cast<v2d*>(&sB[buf][(lc + CPP * q) * LW + 2 * lq]) = rb[q];
    }
  };
  if (nfull > 0) {
    load(kb);
    put(0);
    __syncthreads();
    for (int sl = 0; sl < nfull; ++sl) {
      if (sl + 1 < nfull) load(kb + (int64_t)(sl + 1) * SK);
      __builtin_amdgcn_sched_barrier(0);
      compute(sl & 1);
      __builtin_amdgcn_sched_barrier(0);
      if (sl + 1 < nfull) put((sl + 1) & 1);
      __syncthreads();
    }
  }
  // the wave's two quadrants of tile (tm, tn), in tn_lds_kernel's layout
  const int tm = 2 * tp + wi, tn = 2 * tq + (wj >> 1), ch = wj & 1;
  if (tm >= tilesM || tn >= a.tilesN) return;
  const int tile = tm * a.tilesN + tn;
#pragma unroll
  for (int xh = 0; xh < 2; ++xh) {
    const int quadrant = xh + 2 * ch;
    if (a.nsplit > 1) {
      double* mine = a.part + part_off(split, a.ntiles, tile, quadrant);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int r = 0; r < 4; ++r) mine[((x * 2 + y) * 4 + r) * 64 + lane] = acc[2 * xh + x][y][r];
    } else {
      // one 16 x 16 block at a time (its C2 loads issued before its stores)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int i = tm * 64 + 32 * xh + 16 * x + li;
          const int j0 = tn * 64 + 32 * ch + 16 * y;
          double old[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = j0 + colsub(r, g, false);
            old[r] = (a.C2 && i < a.M2 && j < a.N) ? a.C2[i + (int64_t)j * a.ldc2] : 0.0;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = j0 + colsub(r, g, false);
            const double v = acc[2 * xh + x][y][r];
            if (i < a.M && j < a.N) {
              if (a.C) a.C[i + (int64_t)j * a.ldc] = v;
              if (a.C2 && i < a.M2) a.C2[i + (int64_t)j * a.ldc2] = old[r] + v;
            }
          }
        }
    }
  }
}

// FP32 form of tnq_kernel (the mixed-precision coefficient product
// R_bar = Qbar^T Q_t): 128 x 128 output per 512-thread workgroup, each wave a
// 64 x 32 block.  The operands are rounded to FP32 once, as they are staged,
// and LDS holds FP32 slabs of 32 k-values (72 KB; SK / 2 threads stage one
// column's slab, one 16-byte pair each).  Each 16 k-values are summed in FP32
// on v_mfma_f32_16x16x4_f32 and then added into the FP64 accumulators.  The
// accumulators of both precisions take more than 128 registers: one
// workgroup per CU.  Alone, at K = 49152 with 256 rows and 32768 columns:
// ~93 TFLOP/s, against ~69 when every wave rounded the FP64 operands it read
// from LDS.  K a multiple of 32; output contract of tnq_kernel in the FP32
// result layout.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void tnf_kernel(TnArgs a) {
  constexpr int SK = 32, LW = SK + 4, TPC = SK / 2, CPP = 512 / TPC, NQ = 128 / CPP;
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ float sA[2][128 * LW];
  __shared__ float sB[2][128 * LW];
  const int tilesM = a.ntiles / a.tilesN;
  const int qm = (tilesM + 1) / 2;
  const int tp = blockIdx.x % qm, tq = blockIdx.x / qm, split = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int wi = wave & 1, wj = wave >> 1;
  const int ia0 = 64 * wi, jb0 = 32 * wj;
  const int64_t kb = (int64_t)split * a.kchunk;
  const int64_t ke = std::min<int64_t>(a.K, kb + a.kchunk);
  const int lc = tid / TPC, lq = tid % TPC;
  const double* ga[NQ];
  const double* gb[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = tp * 128 + lc + CPP * q, j = tq * 128 + lc + CPP * q;
    // columns outside the matrix read column 0 and feed only unstored outputs
    ga[q] = a.A + (int64_t)(i < a.M ? i : 0) * a.lda + 2 * lq;
    gb[q] = a.B + (int64_t)(j < a.N ? j : 0) * a.ldb + 2 * lq;
  }
  v4d acc[4][2];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = v4d{0, 0, 0, 0};
  auto compute = [&](int buf) {
    // per 16 k-values: lane group g supplies k-values kk + 4 g .. + 4
#pragma unroll
    for (int kk = 0; kk < SK; kk += 16) {
      v4f t[4][2];
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) t[x][y] = v4f{0, 0, 0, 0};
#pragma unroll
      for (int s0 = 0; s0 < 4; s0 += 2) {
        float fa[4][2], fb[2][2];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const v2f v = *reinterpret_cast<const v2f*>(&sA[buf][(ia0 + 16 * x + li) * LW + kk + 4 * g + s0]);
          fa[x][0] = v.x; fa[x][1] = v.y;
        }
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const v2f v = *reinterpret_cast<const v2f*>(&sB[buf][(jb0 + 16 * y + li) * LW + kk + 4 * g + s0]);
          fb[y][0] = v.x; fb[y][1] = v.y;
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) t[x][y] = mfma(fb[y][s], fa[x][s], t[x][y]);
      }
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) widen_add(acc[x][y], t[x][y]);
    }
  };
  v2d ra[NQ], rb[NQ];
  auto load = [&](int64_t k) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) ra[q] = *reinterpret_cast<const v2d*>(ga[q] + k);
#pragma unroll
    for (int q = 0; q < NQ; ++q) rb[q] = *reinterpret_cast<const v2d*>(gb[q] + k);
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      *reinterpret_cast<v2f*>(&sA[buf][(lc + CPP * q) * LW + 2 * lq]) = v2f{(float)ra[q].x, (float)ra[q].y};
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      *reinterpret_cast<v2f*>(&sB[buf][(lc + CPP * q) * LW + 2 * lq]) = v2f{(float)rb[q].x, (float)rb[q].y};
  };
  const int nfull = (int)((ke - kb) / SK);
  if (nfull > 0) {
    load(kb);
    put(0);
    __syncthreads();
    for (int sl = 0; sl < nfull; ++sl) {
      if (sl + 1 < nfull) load(kb + (int64_t)(sl + 1) * SK);
      __builtin_amdgcn_sched_barrier(0);
      compute(sl & 1);
      __builtin_amdgcn_sched_barrier(0);
      if (sl + 1 < nfull) put((sl + 1) & 1);
      __syncthreads();
    }
  }
  // the wave's two quadrants of tile (tm, tn), in tn_lds_kernel's layout
  const int tm = 2 * tp + wi, tn = 2 * tq + (wj >> 1), ch = wj & 1;
  if (tm >= tilesM || tn >= a.tilesN) return;
  const int tile = tm * a.tilesN + tn;
#pragma unroll
  for (int xh = 0; xh < 2; ++xh) {
    const int quadrant = xh + 2 * ch;
    if (a.nsplit > 1) {
      double* mine = a.part + part_off(split, a.ntiles, tile, quadrant);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int r = 0; r < 4; ++r) mine[((x * 2 + y) * 4 + r) * 64 + lane] = acc[2 * xh + x][y][r];
    } else {
      // one 16 x 16 block at a time (its C2 loads issued before its stores)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int i = tm * 64 + 32 * xh + 16 * x + li;
          const int j0 = tn * 64 + 32 * ch + 16 * y;
          double old[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = j0 + colsub(r, g, true);
            old[r] = (a.C2 && i < a.M2 && j < a.N) ? a.C2[i + (int64_t)j * a.ldc2] : 0.0;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = j0 + colsub(r, g, true);
            const double v = acc[2 * xh + x][y][r];
            if (i < a.M && j < a.N) {
              if (a.C) a.C[i + (int64_t)j * a.ldc] = v;
              if (a.C2 && i < a.M2) a.C2[i + (int64_t)j * a.ldc2] = old[r] + v;
            }
          }
        }
    }
  }
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// x = hi + mid + lo + e with BF16 parts, each the rounding of what the parts
// before it leave (through FP32), |e| <= 2^-26 |x|: the differences x - hi
// and x - hi - mid are exact in FP64 (each part is within a factor 2^-8 of
// what it approximates).
__device__ __forceinline__ void split3(double x, __bf16& h, __bf16& m, __bf16& l) {
  h = (__bf16)(float)x;
  const double r1 = x - (double)(float)h;
  m = (__bf16)(float)r1;
  const double r2 = r1 - (double)(float)m;
  l = (__bf16)(float)r2;
}

// D += X Y on BF16 MFMA, 16 x 16 x 32 (lane l supplies 8 k-values of row l % 16
// of X and of column l % 16 of Y; FP32 result in the f32 layout)
__device__ __forceinline__ v4f mfma_bf(const bf16x8& x, const bf16x8& y, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
}

// Split-BF16 form of tnq_kernel (the mixed-precision coefficient product
// R_bar = Qbar^T Q_t): 128 x 128 output per 512-thread workgroup, each wave a
// 64 x 32 block.  Slabs are 32 deep.  Every staged FP64 element is split
// into three BF16 parts (split3) as it is stored to LDS, into three planes
// per operand (k contiguous, 80-byte column pitch: conflict-free 16-byte
// reads); the product of two elements is taken as the six part products
// whose size is at least 2^-16 of the whole (hi hi, hi mid, mid hi, hi lo,
// lo hi, mid mid; the three dropped ones are below 2^-25 of it), issued
// smallest first into one FP32 accumulator per 32-k slab, which is then
// added into the FP64 accumulators.  Two LDS buffers (120 KB): one
// workgroup per CU, two waves per SIMD.  K a multiple of 32.
template <int TAG>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void tnb_kernel(TnArgs a) {
  constexpr int SK = 32, LW = SK + 8, TPC = SK / 2, CPP = 512 / TPC;   // 16 threads per column, 32 columns a pass
  constexpr int PL = 128 * LW;                                         // one plane of one operand
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ __bf16 sA[2][3 * PL];
  __shared__ __bf16 sB[2][3 * PL];
  const int tilesM = a.ntiles / a.tilesN;
  const int qm = (tilesM + 1) / 2;
  const int tp = blockIdx.x % qm, tq = blockIdx.x / qm, split = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int wi = wave & 1, wj = wave >> 1;
  const int ia0 = 64 * wi, jb0 = 32 * wj;
  const int64_t kb = (int64_t)split * a.kchunk;
  const int64_t ke = std::min<int64_t>(a.K, kb + a.kchunk);
  const int lc = tid / TPC, lq = tid % TPC;
  const double* ga[4];
  const double* gb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = tp * 128 + lc + CPP * q, j = tq * 128 + lc + CPP * q;
    // columns outside the matrix read column 0 and feed only unstored outputs
    ga[q] = a.A + (int64_t)(i < a.M ? i : 0) * a.lda + 2 * lq;
    gb[q] = a.B + (int64_t)(j < a.N ? j : 0) * a.ldb + 2 * lq;
  }
  v4d acc[4][2];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = v4d{0, 0, 0, 0};
  auto compute = [&](int buf) {
    bf16x8 fb[2][3];
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int pl = 0; pl < 3; ++pl)
        fb[y][pl] = *reinterpret_cast<const bf16x8*>(&sB[buf][pl * PL + (jb0 + 16 * y + li) * LW + 8 * g]);
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      bf16x8 fa[3];
#pragma unroll
      for (int pl = 0; pl < 3; ++pl)
        fa[pl] = *reinterpret_cast<const bf16x8*>(&sA[buf][pl * PL + (ia0 + 16 * x + li) * LW + 8 * g]);
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        // issued transposed (B's part first), smallest part products first
        v4f t = v4f{0, 0, 0, 0};
        t = mfma_bf(fb[y][2], fa[0], t);
        t = mfma_bf(fb[y][0], fa[2], t);
        t = mfma_bf(fb[y][1], fa[1], t);
        t = mfma_bf(fb[y][1], fa[0], t);
        t = mfma_bf(fb[y][0], fa[1], t);
        t = mfma_bf(fb[y][0], fa[0], t);
        widen_add(acc[x][y], t);
      }
    }
  };
  const int nsl = (int)((ke - kb) / SK);
  v2d ra[4], rb[4];
  auto load = [&](int64_t k) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ra[q] = *reinterpret_cast<const v2d*>(ga[q] + k);
      rb[q] = *reinterpret_cast<const v2d*>(gb[q] + k);
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      __bf16 h0, m0, l0, h1, m1, l1;
      const int off = (lc + CPP * q) * LW + 2 * lq;
      split3(ra[q].x, h0, m0, l0);
      split3(ra[q].y, h1, m1, l1);
      *reinterpret_cast<bf16x2*>(&sA[buf][off]) = bf16x2{h0, h1};
      *reinterpret_cast<bf16x2*>(&sA[buf][PL + off]) = bf16x2{m0, m1};
      *reinterpret_cast<bf16x2*>(&sA[buf][2 * PL + off]) = bf16x2{l0, l1};
      split3(rb[q].x, h0, m0, l0);
      split3(rb[q].y, h1, m1, l1);
      *reinterpret_cast<bf16x2*>(&sB[buf][off]) = bf16x2{h0, h1};
      *reinterpret_cast<bf16x2*>(&sB[buf][PL + off]) = bf16x2{m0, m1};
      *reinterpret_cast<bf16x2*>(&sB[buf][2 * PL + off]) = bf16x2{l0, l1};
    }
  };
  if (nsl > 0) {
    load(kb);
    put(0);
    __syncthreads();
    for (int sl = 0; sl < nsl; ++sl) {
      if (sl + 1 < nsl) load(kb + (int64_t)(sl + 1) * SK);
      __builtin_amdgcn_sched_barrier(0);
      compute(sl & 1);
      __builtin_amdgcn_sched_barrier(0);
      if (sl + 1 < nsl) put((sl + 1) & 1);
      __syncthreads();
    }
  }
  // the wave's two quadrants of tile (tm, tn), in tn_lds_kernel's layout (f32 form)
  const int tm = 2 * tp + wi, tn = 2 * tq + (wj >> 1), ch = wj & 1;
  if (tm >= tilesM || tn >= a.tilesN) return;
  const int tile = tm * a.tilesN + tn;
#pragma unroll
  for (int xh = 0; xh < 2; ++xh) {
    const int quadrant = xh + 2 * ch;
    if (a.nsplit > 1) {
      double* mine = a.part + part_off(split, a.ntiles, tile, quadrant);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int r = 0; r < 4; ++r) mine[((x * 2 + y) * 4 + r) * 64 + lane] = acc[2 * xh + x][y][r];
    } else {
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int i = tm * 64 + 32 * xh + 16 * x + li;
          const int j0 = tn * 64 + 32 * ch + 16 * y;
          double old[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = j0 + colsub(r, g, true);
            old[r] = (a.C2 && i < a.M2 && j < a.N) ? a.C2[i + (int64_t)j * a.ldc2] : 0.0;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = j0 + colsub(r, g, true);
            const double v = acc[2 * xh + x][y][r];
            if (i < a.M && j < a.N) {
              if (a.C) a.C[i + (int64_t)j * a.ldc] = v;
              if (a.C2 && i < a.M2) a.C2[i + (int64_t)j * a.ldc2] = old[r] + v;
            }
          }
        }
    }
  }
}

// Fallback for operands that are not 16-byte aligned or have odd leading
// dimensions: direct scalar loads, same tiling and output contract.
__global__ __launch_bounds__(256) void tn_direct_kernel(TnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  const int tile = blockIdx.x, split = blockIdx.y;
  const int tm = tile / a.tilesN, tn = tile % a.tilesN;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int i0 = tm * 64 + (wave & 1) * 32, j0 = tn * 64 + (wave >> 1) * 32;
  const int64_t kb = (int64_t)split * a.kchunk;
  const int64_t ke = std::min<int64_t>(a.K, kb + a.kchunk);
  const double* ap[2];
  const double* bp[2];
  bool aok[2], bok[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    int i = i0 + 16 * t + li, j = j0 + 16 * t + li;
    aok[t] = i < a.M;
    bok[t] = j < a.N;
    ap[t] = a.A + (int64_t)(aok[t] ? i : 0) * a.lda;
    bp[t] = a.B + (int64_t)(bok[t] ? j : 0) * a.ldb;
  }
  v4d acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = v4d{0, 0, 0, 0};
  for (int64_t k0 = kb; k0 < ke; k0 += 16) {
    double xa[2][4], xb[2][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int64_t k = k0 + 4 * g + s;
      const bool kok = k < ke;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        xa[t][s] = (aok[t] && kok) ? ap[t][k] : 0.0;
        xb[t][s] = (bok[t] && kok) ? bp[t][k] : 0.0;
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = mfma(xb[y][s], xa[x][s], acc[x][y]);
  }
  tn_store(a, acc, tile, split, wave, lane, i0, j0, false);
}

// --------------------------------------------------------------------------
// The same product where 64 x 64 tiles would leave the chip idle: a panel of a
// small matrix has a few such tiles, and a depth too short to split, so a few
// compute units would do all of the work behind their matrix cores (a 16-column
// panel of 320 rows: 5 tiles of 10 slabs, 16 us, of which most is padding of
// 16 columns to 64).  Here a workgroup forms 16 x 16 outputs and its 16 waves
// share the depth, 16 k-values at a time in turn, straight from memory (the
// operands of such products are in cache), two chunks ahead; the
// waves' sums are added through LDS in order, so there are no partials and no
// second launch.
// --------------------------------------------------------------------------

constexpr int kSmallWaves = 16;
// A workgroup reads its 32 columns at some 40-70 GB/s, so the depth it can take
// is short: at 2304 rows the split product and its reduction are as fast (one
// tile: 17.4 us and 5 against 17.3), at 4608 faster (17.5 and 5 against 32.6).
// From two workgroups per CU on the 64 x 64 tiles' fewer reads win (1386 rows x
// 16 x 4096: 256 of them, 33 us against 12; x 64 x 4096: 33 against 43).
constexpr int64_t kSmallDepth = 2048;
constexpr int64_t kSmallGrid = 512;

template <int TAG, bool VEC>
__global__ __launch_bounds__(64 * kSmallWaves) void tns_kernel(TnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ double red[kSmallWaves][4][64];
  const int tilesM = (a.M + 15) / 16;
  const int i0 = blockIdx.x % tilesM * 16, j0 = blockIdx.x / tilesM * 16;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // columns outside the matrix read column 0 and feed only unstored outputs
  // lane group g holds k-values 2g, 2g + 1, 8 + 2g, 9 + 2g of a chunk: a load
  // takes 64 contiguous bytes of each column
  const double* pa = a.A + (int64_t)(i0 + li < a.M ? i0 + li : 0) * a.lda + 2 * g;
  const double* pb = a.B + (int64_t)(j0 + li < a.N ? j0 + li : 0) * a.ldb + 2 * g;
  const int nfull = (int)(a.K / 16);
  const int mine = (nfull - wave + kSmallWaves - 1) / kSmallWaves;      // the wave's whole chunks
  v4d acc = v4d{0, 0, 0, 0};
  double x0[8], x1[8], y0[8], y1[8];
  auto load = [&](double (&x)[8], int q) {
    const int64_t k = 16 * (int64_t)(wave + q * kSmallWaves);
    if constexpr (VEC) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const v2d u = *reinterpret_cast<const v2d*>(pa + k + 8 * h), v = *reinterpret_cast<const v2d*>(pb + k + 8 * h);
        x[2 * h] = u.x; x[2 * h + 1] = u.y; x[4 + 2 * h] = v.x; x[5 + 2 * h] = v.y;
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        x[s] = pa[k + (s & 1) + 4 * (s & 2)];
        x[4 + s] = pb[k + (s & 1) + 4 * (s & 2)];
      }
    }
  };
  auto mac = [&](const double (&x)[8]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = mfma(x[4 + s], x[s], acc);
  };
  if (mine > 0) load(x0, 0);
  if (mine > 1) load(x1, 1);
#pragma unroll 1
  for (int q = 0; q < mine; q += 4) {
    if (q + 2 < mine) load(y0, q + 2);
    if (q + 3 < mine) load(y1, q + 3);
    mac(x0);
    if (q + 1 < mine) mac(x1);
    if (q + 4 < mine) load(x0, q + 4);
    if (q + 5 < mine) load(x1, q + 5);
    if (q + 2 < mine) mac(y0);
    if (q + 3 < mine) mac(y1);
  }
  if (const int64_t k0 = 16 * (int64_t)nfull; k0 < a.K && wave == nfull % kSmallWaves) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int64_t k = k0 + (s & 1) + 4 * (s & 2);
      const bool in = k + 2 * g < a.K;
      x0[s] = in ? pa[k] : 0.0;
      x0[4 + s] = in ? pb[k] : 0.0;
    }
    mac(x0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][r][lane] = acc[r];
  __syncthreads();
  if (tid >= 256) return;
  const int i = i0 + li, j = j0 + 4 * wave + g;              // element r = wave of the waves' accumulators
  double v = 0.0;
#pragma unroll
  for (int e = 0; e < kSmallWaves; ++e) v += red[e][wave][lane];
  if (i >= a.M || j >= a.N) return;
  if (a.C) a.C[i + (int64_t)j * a.ldc] = v;
  if (a.C2 && i < a.M2) a.C2[i + (int64_t)j * a.ldc2] += v;
}

// Sum the split partials in split order; write C (and C2 +=).  A workgroup of G
// groups of 64 threads takes U of a wave quadrant's 16 element slots per lane;
// each group sums a contiguous range of the splits and the groups' sums are
// added in order.  Bound by reading the partials: few output tiles and many
// splits (a Gram product of a tall matrix: one tile, 288 splits) would
// otherwise leave 4 workgroups a tile reading them one after the other.
template <int G, int U>
__global__ __launch_bounds__(64 * G) void tn_reduce_split_kernel(TnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ double red[G][U][64];
  constexpr int kSlots = 16 / U;               // workgroups per quadrant
  const int tile = blockIdx.x / (4 * kSlots), wave = blockIdx.x / kSlots & 3, q0 = blockIdx.x % kSlots * U;
  const int tm = tile / a.tilesN, tn = tile % a.tilesN;
  if (a.lower && (tn >> 1) > (tm >> 1)) return;
  const int grp = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  // the element this thread finishes: slot q = q0 + grp (groups below U)
  const int q = q0 + grp % U;
  const int i = tm * 64 + (wave & 1) * 32 + 16 * (q >> 3) + li;
  const int j = tn * 64 + (wave >> 1) * 32 + 16 * (q >> 2 & 1) + colsub(q & 3, g, a.f32);
  const bool out = grp < U && i < a.M && j < a.N;
  const bool add = out && a.C2 && i < a.M2;
  const double old = add ? a.C2[i + (int64_t)j * a.ldc2] : 0.0;
  const int per = (a.nsplit + G - 1) / G, s0 = grp * per, s1 = std::min(a.nsplit, s0 + per);
  const double* base = a.part + part_off(0, a.ntiles, tile, wave) + q0 * 64 + lane;
  const int64_t sstride = (int64_t)a.ntiles * 4 * 1024;
  double v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = 0.0;
  for (int sp0 = s0; sp0 < s1; sp0 += 16) {
    double t[16][U];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int sp = std::min(sp0 + k, s1 - 1);         // clamped: extra loads are discarded
#pragma unroll
      for (int u = 0; u < U; ++u) t[k][u] = base[sp * sstride + u * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 16; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] += sp0 + k < s1 ? t[k][u] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) red[grp][u][lane] = v[u];
  __syncthreads();
  if (!out) return;
  double x = 0.0;
#pragma unroll
  for (int e = 0; e < G; ++e) x += red[e][grp][lane];
  if (a.C) a.C[i + (int64_t)j * a.ldc] = x;
  if (add) a.C2[i + (int64_t)j * a.ldc2] = old + x;
}

// The same for few splits: one block per wave quadrant of a tile, thread
// (qg, lane) owns 4 of the lane's 16 values and sums all splits.
__global__ __launch_bounds__(256) void tn_reduce_kernel(TnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  const int tile = blockIdx.x >> 2, wave = blockIdx.x & 3;
  const int tm = tile / a.tilesN, tn = tile % a.tilesN;
  if (a.lower && (tn >> 1) > (tm >> 1)) return;
  const int qg = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int i = tm * 64 + (wave & 1) * 32 + 16 * (qg >> 1) + li;
  const int jq = tn * 64 + (wave >> 1) * 32 + 16 * (qg & 1);         // + colsub(u, g)
  double old[4];
  if (a.C2) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = jq + colsub(u, g, a.f32);
      old[u] = (i < a.M2 && j < a.N) ? a.C2[i + (int64_t)j * a.ldc2] : 0.0;
    }
  }
  double v[4];
  sum_partials4(a.part, a.nsplit, a.ntiles, tile, wave, qg, lane, v);
  if (i >= a.M) return;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = jq + colsub(u, g, a.f32);
    if (j < a.N) {
      if (a.C) a.C[i + (int64_t)j * a.ldc] = v[u];
      if (a.C2 && i < a.M2) a.C2[i + (int64_t)j * a.ldc2] = old[u] + v[u];
    }
  }
}

static bool aligned16(const void* p, int64_t ld) {
  return (reinterpret_cast<uintptr_t>(p) % 16 == 0) && (ld % 2 == 0);
}

static int pick_split(int tiles, int64_t K, int64_t cap, int64_t rows) {
  // Below 256 workgroups: at most 512 (two resident per CU, so one wave of
  // workgroups; a few over that run as a second wave and cost ~16% at 79
  // tiles).  From 256 on, splits up to ~1280 workgroups: the shorter
  // workgroups even out the last wave (alone, the 128 x 20480 product with
  // depth 24576 runs at 51.6 TFLOP/s with two splits against 44.3 with one).
  // Each split keeps at least `rows` rows.
  int want = tiles >= 256 ? (1280 + tiles - 1) / tiles : std::max(1, 512 / std::max(1, tiles));
  int64_t maxs = std::max<int64_t>(1, K / rows);
  int ns = (int)std::min<int64_t>(want, maxs);
  while (ns > 1 && (int64_t)ns * tiles > cap) --ns;
  return ns;
}

// The 512-thread products (128 x 128 or two-tile-row; two workgroups per CU,
// 512 slots): about 1280 workgroups whatever the tile count, so that the last
// wave of workgroups is short, each split keeping at least `rows` rows.  Alone, the 128 x 20480
// product of depth 24576 (160 tiles) runs at 60.8 TFLOP/s with 8 splits
// against 51.5 with the 3 that filling one wave of slots gives.
static int pick_split_quad(int blocks, int64_t K, int64_t cap, int tiles, int64_t rows = 256) {
  const int64_t maxs = std::max<int64_t>(1, K / rows);
  int ns = (int)std::min<int64_t>((1280 + blocks - 1) / blocks, maxs);
  while (ns > 1 && (int64_t)ns * tiles > cap) --ns;
  return std::max(ns, 1);
}

// The 128 x 128 products of short duration: as many workgroups as half the slots
// or all of them (512) hold, where those divide well among the blocks, so a
// fraction of the partials of 1280 (us, product and sum, 1280, 512 and 256
// workgroups: 512 x 512 x 5120: 82, 63, 57; 128 x 4096 x 5120: 129, 101, 101;
// 512 x 512 x 20480: 212, 180, 184).  Longer ones stay with 1280: beside the
// panel chain the n = 16384 factorization loses 0.8% with 512.
static int pick_split_wave(int blocks, int64_t K, int64_t cap, int tiles) {
  if (blocks * K > 350000) return pick_split_quad(blocks, K, cap, tiles);
  const int slots = blocks * K <= 90000 ? 256 : 512;
  int ns = (int)std::min<int64_t>(slots / blocks, K / 64);
  if (blocks * ns < slots - slots / 10 && blocks * (K / 64) > slots) return pick_split_quad(blocks, K, cap, tiles);
  while (ns > 1 && (int64_t)ns * tiles > cap) --ns;
  return std::max(ns, 1);
}

// Least rows of a split: 256 (8 slabs), so that a split's partials stay small
// against its operands; fewer where the whole product leaves the GPU idle, as
// long as it stays below a workgroup per CU (us, product and sum; splits of
// 256, 128 and 64 rows; 64 x 64 x 2304: 17.7, 13.2, 11.7; x 9216: 18.1, 12.6,
// 11.9; x 20480: 17.5, 13.8, 17.7; 512 x 64 x 2304: 18.4, 14.9, 17.2; 1024 x 64 x
// 2304: 19.6, 21.1, 23.4).
static int64_t split_rows(int64_t blocks, int64_t K) {
  return blocks * (K / 64) <= 224 ? 64 : blocks * (K / 128) <= 256 ? 128 : 256;
}

TnArgs tn_setup(const double* A, int64_t lda, const double* B, int64_t ldb, int M, int N, int64_t K, double* C,
                int64_t ldc, double* C2, int64_t ldc2, const Scratch& s, int force_split, int lowp, bool fine) {
  const bool f32 = lowp != 0;
  TnArgs a{};
  a.A = A; a.lda = lda; a.B = B; a.ldb = ldb;
  a.C = C; a.ldc = ldc; a.C2 = C2; a.ldc2 = ldc2; a.M2 = M;
  const int tilesM = (M + kTile - 1) / kTile, tilesN = (N + kTile - 1) / kTile;
  const int tiles = tilesM * tilesN;
  const bool vec = aligned16(A, lda) && aligned16(B, ldb);
  // two tile rows per workgroup from two tile rows and four tile columns on
  // (with fewer tile columns the re-projections on the panel chain slow down)
  const bool pair = vec && tilesM >= 2 && tilesN >= 4;
  // products of at least two tile rows and columns: 128 x 128 per workgroup
  // and a depth that is a multiple of 16 (whole slabs in every split)
  // (32 for FP32 products, whose slabs are 32 deep)
  // (fine: small ones are better spread over 64 x 64 tiles, 128 x 128 x 5120: 16
  // us against 20, 512 x 128 x 2304: 21 and 27, x 5120: 31 and 26)
  const bool quad = vec && tilesM >= 2 && tilesN >= 2 && K % (f32 ? 32 : 16) == 0 && !(fine && tiles * K <= 40000);
  // the split-BF16 product on the same 128 x 128 tiles
  const bool bf3 = vec && lowp == 2 && tilesM >= 2 && tilesN >= 2 && K % 32 == 0;
  // the split count fills the grid of workgroups the product launches
  const int blocks = quad || bf3 ? (tilesM + 1) / 2 * ((tilesN + 1) / 2) : pair ? (tilesM + 1) / 2 * tilesN : tiles;
  const int64_t rows = fine ? split_rows(blocks, K) : 256;
  int ns = force_split > 0 ? force_split
           : quad && fine        ? pick_split_wave(blocks, K, s.npart, tiles)
           : quad || bf3 || pair ? pick_split_quad(blocks, K, s.npart, tiles, rows)
                           : pick_split(blocks, K, s.npart, rows);
  while (ns > 1 && (int64_t)ns * tiles > s.npart) --ns;
  int64_t kchunk = (K + ns - 1) / ns;
  kchunk = (kchunk + KC - 1) / KC * KC;
  ns = (int)((K + kchunk - 1) / kchunk);
  a.M = M; a.N = N; a.K = K; a.kchunk = kchunk; a.nsplit = ns; a.tilesN = tilesN; a.ntiles = tiles;
  a.part = s.part;
  a.vec = vec;
  a.f32 = f32 && a.vec;     // the FP32 form exists for the LDS-staged kernel
  a.pair = pair && !quad && !bf3;
  a.quad = quad;
  a.bf3 = bf3;
  return a;
}

// A square product of which only the lower triangle is read: the 128 x 128
// kernel leaves the blocks above the diagonal out (the others compute all of
// C), which halves its work.  Split as pick_split_quad does, for the blocks
// that run.  The grid holds only those: empty workgroups in a full grid would
// leave the XCDs, which take workgroups in turn, with unequal shares.
TnArgs tn_setup_lower(const double* A, int64_t lda, const double* B, int64_t ldb, int N, int64_t K, double* C,
                      int64_t ldc, const Scratch& s) {
  const int t = (N + 2 * kTile - 1) / (2 * kTile), tiles = (N + kTile - 1) / kTile;
  const int ns = pick_split_wave(t * (t + 1) / 2, K, s.npart, tiles * tiles);
  TnArgs a = tn_setup(A, lda, B, ldb, N, N, K, C, ldc, nullptr, 0, s, 0, 0, true);
  if (!a.quad) return a;
  a = tn_setup(A, lda, B, ldb, N, N, K, C, ldc, nullptr, 0, s, ns, 0, true);
  a.lower = 1;
  return a;
}

bool tn_small(TnArgs& a) {
  const int64_t wgs = ((int64_t)a.M + 15) / 16 * ((a.N + 15) / 16);
  if (a.f32 || a.bf3 || a.K > kSmallDepth || wgs > kSmallGrid) return false;
  a.small = 1;
  a.nsplit = 1;
  a.lower = 0;
  return true;
}

template <bool VEC>
static void launch_tns_as(const TnArgs& a, dim3 grid, int tag, hipStream_t st) {
  const dim3 threads(64 * kSmallWaves);
  switch (tag) {
    case TAG_TRAIL: hipLaunchKernelGGL((tns_kernel<TAG_TRAIL, VEC>), grid, threads, 0, st, a); break;
    case TAG_REPROJ: hipLaunchKernelGGL((tns_kernel<TAG_REPROJ, VEC>), grid, threads, 0, st, a); break;
    default: hipLaunchKernelGGL((tns_kernel<TAG_PANEL, VEC>), grid, threads, 0, st, a); break;
  }
}

static void launch_tns(const TnArgs& a, dim3 grid, int tag, hipStream_t st) {
  if (a.vec)
    launch_tns_as<true>(a, grid, tag, st);
  else
    launch_tns_as<false>(a, grid, tag, st);
}

void launch_tn_product(const TnArgs& a, int tag, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0) return;
  if (a.small) {
    const dim3 grids((unsigned)((a.M + 15) / 16 * ((a.N + 15) / 16)));
    launch_tns(a, grids, tag, st);
    return;
  }
  const dim3 grid(a.ntiles, a.nsplit);
  if (!a.vec) {
    hipLaunchKernelGGL(tn_direct_kernel, grid, dim3(256), 0, st, a);
    return;
  }
  if (a.bf3) {
    const dim3 gridb((unsigned)((a.ntiles / a.tilesN + 1) / 2 * ((a.tilesN + 1) / 2)), a.nsplit);
    hipLaunchKernelGGL((tnb_kernel<TAG_TRAIL>), gridb, dim3(512), 0, st, a);
    return;
  }
  if (a.quad) {
    const unsigned qm = (a.ntiles / a.tilesN + 1) / 2, qn = (a.tilesN + 1) / 2;
    const dim3 gridq(a.lower ? qm * (qm + 1) / 2 : qm * qn, a.nsplit);
    if (a.f32) {
      hipLaunchKernelGGL(tnf_kernel, gridq, dim3(512), 0, st, a);
      return;
    }
    switch (tag) {
      case TAG_TRAIL: hipLaunchKernelGGL((tnq_kernel<TAG_TRAIL>), gridq, dim3(512), 0, st, a); break;
      case TAG_REPROJ: hipLaunchKernelGGL((tnq_kernel<TAG_REPROJ>), gridq, dim3(512), 0, st, a); break;
      default: hipLaunchKernelGGL((tnq_kernel<TAG_PANEL>), gridq, dim3(512), 0, st, a); break;
    }
    return;
  }
  if (a.pair) {
    const dim3 grid2((unsigned)((a.ntiles / a.tilesN + 1) / 2 * a.tilesN), a.nsplit);
    if (a.f32) {
      hipLaunchKernelGGL((tn2_kernel<TAG_TRAIL, true>), grid2, dim3(512), 0, st, a);
      return;
    }
    switch (tag) {
      case TAG_TRAIL: hipLaunchKernelGGL((tn2_kernel<TAG_TRAIL, false>), grid2, dim3(512), 0, st, a); break;
      case TAG_REPROJ: hipLaunchKernelGGL((tn2_kernel<TAG_REPROJ, false>), grid2, dim3(512), 0, st, a); break;
      default: hipLaunchKernelGGL((tn2_kernel<TAG_PANEL, false>), grid2, dim3(512), 0, st, a); break;
    }
    return;
  }
  if (a.f32 && a.ntiles / a.tilesN >= 2 && a.tilesN >= 2) {
    hipLaunchKernelGGL((tn16_kernel<TAG_TRAIL, true>), grid, dim3(256), 0, st, a);
    return;
  }
  if (a.f32) {
    hipLaunchKernelGGL((tn_lds_kernel<TAG_TRAIL, true>), grid, dim3(256), 0, st, a);
    return;
  }
  switch (tag) {
    case TAG_TRAIL: hipLaunchKernelGGL((tn_lds_kernel<TAG_TRAIL, false>), grid, dim3(256), 0, st, a); break;
    case TAG_REPROJ: hipLaunchKernelGGL((tn_lds_kernel<TAG_REPROJ, false>), grid, dim3(256), 0, st, a); break;
    default: hipLaunchKernelGGL((tn_lds_kernel<TAG_PANEL, false>), grid, dim3(256), 0, st, a); break;
  }
}

static void launch_tn_sum(const TnArgs& a, hipStream_t st) {
  // one batch of 16 loads per thread covers up to 16 splits; beyond that the
  // splits are shared by 4 or 16 groups of threads, or (seq) only the elements
  // by more workgroups
  if (a.seq && a.nsplit > 16)
    hipLaunchKernelGGL((tn_reduce_split_kernel<1, 1>), dim3(a.ntiles * 64), dim3(64), 0, st, a);
  else if (a.nsplit <= 16)
    hipLaunchKernelGGL(tn_reduce_kernel, dim3(a.ntiles * 4), dim3(256), 0, st, a);
  else if (a.nsplit <= 64)
    hipLaunchKernelGGL((tn_reduce_split_kernel<4, 4>), dim3(a.ntiles * 16), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((tn_reduce_split_kernel<16, 1>), dim3(a.ntiles * 64), dim3(1024), 0, st, a);
}

void launch_tn_reduce(const TnArgs& a, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0 || a.nsplit <= 1) return;
  launch_tn_sum(a, st);
}

// --------------------------------------------------------------------------
// Upper Cholesky factor of a panel leaf's Gram matrix W (w <= kLeaf), its
// inverse, and on the second pass R2 R1 and the lookahead coefficients T^T X.
// One block of four waves (see chol_blocked for the factorization).  A
// pivot at most kCholBreak times its column's diagonal entry is a breakdown,
// handled by the column-wise fallback described at panel_second_kernel.
// --------------------------------------------------------------------------

// Smallest pivot / diagonal ratio a Cholesky-QR pass accepts: below it a
// column lies within 1e-7 rad of the span of the columns before it, the
// panel's condition number exceeds ~1e7, and one Cholesky-QR pass could no
// longer bring the panel close enough to orthonormal for the second to finish.
constexpr double kCholBreak = 1e-14;


// 1/sqrt(x) to full double precision: hardware estimate plus one Newton step.
__device__ __forceinline__ double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x * y;
  const double r = fma(-h, y, 0.5);
  return fma(y, r, y);
}

// One wave factors the 16 x 16 diagonal block at offset o of Rl (its upper
// triangle, already updated, read symmetrically): Gauss elimination of the
// augmented [D | I] with each final row scaled by 1/sqrt(pivot), so D = R^T R
// gives R (into Rl's block, zero below the diagonal) and T = R^{-1} (into
// Tl's block).  Lanes 0..15 hold column tx of D, lanes 16..31 column tx of
// the identity half, 16 rows in registers.  Step j: row j of D (by symmetry
// also column j) lies in the D lanes' register j; every lane takes the pivot
// and the column-j factors from there by readlane, and subtracts.  A serial
// chain of 16 steps, bound by the latency of each: through LDS, with the
// results stored as they came, a 64-column factorization took 31 us of its
// kernel's 35, so 20 of 25.
__device__ __forceinline__ void chol_diag16(int lane, int o, double (*Rl)[kLeaf + 1], double (*Tl)[kLeaf + 1],
                                            const double* dg, bool& bad) {
  const int tx = lane & 15;
  const bool dl = lane < 16, zl = lane >= 16 && lane < 32;
  // lane l's value in every lane
  auto from = [](double x, int l) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
  };
  double c[16];
#pragma unroll
  for (int i = 0; i < 16; ++i)
    c[i] = dl ? ((i <= tx) ? Rl[o + i][o + tx] : Rl[o + tx][o + i]) : (zl && i == tx ? 1.0 : 0.0);
  const double least = kCholBreak * dg[o + tx];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    // breakdown: a pivot that is not positive, or below kCholBreak times the
    // column's diagonal entry in the Gram matrix (the column lies within an
    // angle of 1e-7 of the span of the columns before it)
    double piv = from(c[j], j);
    const bool ok = piv > from(least, j) && isfinite(piv);
    bad |= !ok;
    piv = ok ? piv : 1.0;
    const double inv = rsqrt_nr(piv);
    const double r = c[j] * inv, f = r * inv;
#pragma unroll
    for (int i = j + 1; i < 16; ++i) c[i] -= from(c[j], i) * f;
    c[j] = r;
    // (each step's updates before the next step: left to itself the compiler
    // keeps the factors of all steps in scalar registers, spills them, and
    // updates each row when it is needed, in one long chain)
#pragma unroll
    for (int i = j + 1; i < 16; ++i) asm volatile("" : "+v"(c[i]));
  }
  if (dl) {
#pragma unroll
    for (int j = 0; j < 16; ++j) Rl[o + j][o + tx] = (tx >= j) ? c[j] : 0.0;
  } else if (zl) {
#pragma unroll
    for (int j = 0; j < 16; ++j) Tl[o + tx][o + j] = c[j];
  }
}

// Exact path: blocked right-looking Cholesky of W (16 nb columns, nb <= 4) in
// Rl (16 x 16 blocks) and the inverse T = R^{-1} in Tl, which comes in as the
// identity.  Block step b: wave 0 factors the diagonal block (R_bb, T_bb); the
// row panel R_bc = T_bb^T W_bc (c > b) and the trailing update W_cd -= R_bc^T
// R_bd (b < c <= d) run on MFMA, one 16 x 16 block per wave.  Then T's
// off-diagonal blocks, one block column per wave: T_ab = -T_aa sum_{c=a+1..b}
// R_ac T_cb for a = b-1 down to 0.  About three block barriers per 16 columns.
__device__ __forceinline__ void chol_blocked(int tid, int nb, double (*Rl)[kLeaf + 1], double (*Tl)[kLeaf + 1],
                                             const double* dg, bool& bad) {
  const int wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
#pragma unroll 1
  for (int b = 0; b < nb; ++b) {
    const int o = 16 * b;
    if (wave == 0) chol_diag16(lane, o, Rl, Tl, dg, bad);
    __syncthreads();
    if (b + 1 == nb) break;
    // row panel R_bc = T_bb^T W_bc, in place
    const int c = b + 1 + wave;
    if (c < nb) {
      v4d acc = v4d{0, 0, 0, 0};
      mma16(acc, lane, 1, [&](int i, int k) { return Tl[o + k][o + i]; },
            [&](int k, int j) { return Rl[o + k][16 * c + j]; });
#pragma unroll
      for (int r = 0; r < 4; ++r) Rl[o + li][16 * c + 4 * r + g] = acc[r];
    }
    __syncthreads();
    // trailing update W_cd -= R_bc^T R_bd over the upper blocks b < c <= d
    int p = 0;
#pragma unroll 1
    for (int cc = b + 1; cc < nb; ++cc)
#pragma unroll 1
      for (int dd = cc; dd < nb; ++dd, ++p) {
        if ((p & 3) != wave) continue;
        v4d acc = v4d{0, 0, 0, 0};
        mma16(acc, lane, 1, [&](int i, int k) { return Rl[o + k][16 * cc + i]; },
              [&](int k, int j) { return Rl[o + k][16 * dd + j]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) Rl[16 * cc + li][16 * dd + 4 * r + g] -= acc[r];
      }
    __syncthreads();
  }
  // block column wave of T (the blocks below the diagonal are zero in T as it
  // comes in, and zeroed in R here: the columns left of block row `wave`)
#pragma unroll 1
  for (int a = wave < nb ? wave - 1 : -1; a >= 0; --a) {
    v4d acc = v4d{0, 0, 0, 0};
#pragma unroll 1
    for (int cb = a + 1; cb <= wave; ++cb)
      mma16(acc, lane, 1, [&](int i, int k) { return Rl[16 * a + i][16 * cb + k]; },
            [&](int k, int j) { return Tl[16 * cb + k][16 * wave + j]; });
#pragma unroll
    for (int r = 0; r < 4; ++r) Tl[16 * a + li][16 * wave + 4 * r + g] = acc[r];
    __builtin_amdgcn_wave_barrier();
    v4d t = v4d{0, 0, 0, 0};
    mma16(t, lane, 1, [&](int i, int k) { return Tl[16 * a + i][16 * a + k]; },
          [&](int k, int j) { return Tl[16 * a + k][16 * wave + j]; });
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r) Tl[16 * a + li][16 * wave + 4 * r + g] = -t[r];
    __builtin_amdgcn_wave_barrier();
  }
  for (int e = lane; e < 16 * 16 * wave; e += 64) Rl[16 * wave + (e & 15)][e >> 4] = 0.0;
  __syncthreads();
}

// C = A B for upper triangular w x w LDS matrices (row-major, 64 x 64 with
// identity padding; C[i][j] needs only k in [i, j]: k blocks left of the row
// block are skipped).  Wave v computes rows 16v..16v+15 and stores C into the
// column-major global matrix out (ld ldo).
__device__ __forceinline__ void lds_mm_store(int tid, const double (*Al)[kLeaf + 1], const double (*Bl)[kLeaf + 1],
                                             int w, double* out, int64_t ldo) {
  const int wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  v4d acc[4];
#pragma unroll
  for (int y = 0; y < 4; ++y) acc[y] = v4d{0, 0, 0, 0};
  for (int k0 = 16 * wave; k0 < w; k0 += 16) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + 4 * g + s;
      const double xa = Al[16 * wave + li][k];
#pragma unroll
      for (int y = 0; y < 4; ++y)
        if (16 * y < w) acc[y] = mfma(Bl[k][16 * y + li], xa, acc[y]);
    }
  }
  const int i = 16 * wave + li;
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = 16 * y + 4 * r + g;
      if (i < w && j < w) out[i + (int64_t)j * ldo] = acc[y][r];
    }
}

// The split reduction of a trailing-update product W = P1^T Q_t formed from
// a panel after its first Cholesky pass, with the second pass's transform
// folded in: out = T^T W (T = R2^{-1}, w x w upper triangular) equals
// (P1 T)^T Q_t, the coefficients against the finished panel P = P1 T.  M = w
// <= 64, so the product has a single tile row; four blocks share a 64-column
// tile, block cg taking the 16 columns that two wave quadrants of the product
// hold in their accumulator registers (quadrant column half cg >> 1, lane
// column group cg & 1).  The 64 x 16 strip of W is summed in split order into
// LDS (or read from a.C, where a product without a split stored it) and
// multiplied by T^T on MFMA, wave v forming rows 16v .. 16v + 15.
// When the panel's second pass took the column-wise fallback (*fb set), the
// finished panel is no longer P1 T, and the strip's coefficients are formed
// directly as P^T Q_t over the a.K rows (P: ld ldp, Q_t = a.B), on MFMA with
// operands read straight from memory (a rare path; its speed does not
// matter).
__global__ __launch_bounds__(256) void tn_reduce_tmul_kernel(TnArgs a, const double* T, int w, double* out,
                                                             int64_t ldo, const int* fb, const double* P,
                                                             int64_t ldp) {
  __shared__ double Wl[kLeaf][16 + 1];
  __shared__ double Tl[kLeaf][kLeaf + 1];
  const int tile = blockIdx.x >> 2, cg = blockIdx.x & 3, tid = threadIdx.x;
  const int lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int64_t jc = (int64_t)tile * kTile + (cg >> 1) * 32 + 16 * (cg & 1);   // first column of the strip
  const int wc = (int)std::max<int64_t>(0, std::min<int64_t>(16, a.N - jc));
  if (fb && *fb) {
    const int wave = tid >> 6;
    const int i = 16 * wave + li, j = li;
    const double* pa = P + (int64_t)(i < w ? i : 0) * ldp;
    const double* pb = a.B + (jc + (j < wc ? j : 0)) * a.ldb;
    v4d acc = v4d{0, 0, 0, 0};
    for (int64_t k0 = 0; k0 < a.K; k0 += 16) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int64_t k = k0 + 4 * g + s;
        const double xa = (k < a.K && i < w) ? pa[k] : 0.0;
        const double xb = (k < a.K && j < wc) ? pb[k] : 0.0;
        acc = mfma(xb, xa, acc);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int jj = 4 * r + g;
      if (i < w && jj < wc) out[i + (jc + jj) * ldo] = acc[r];
    }
    return;
  }
  double tv[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int e = tid + 256 * q, k = e & 63, i = e >> 6;
    tv[q] = (k < w && i < w) ? T[k + (int64_t)i * w] : 0.0;
  }
  if (a.nsplit > 1) {
    // thread (row half wr, row group qh, lane) sums 4 values of quadrant
    // wr + 2 (cg >> 1), lane group 2 qh + (cg & 1)
    const int wr = tid >> 7, qh = (tid >> 6) & 1;
    double v[4];
    sum_partials4(a.part, a.nsplit, a.ntiles, tile, wr | ((cg >> 1) << 1), (qh << 1) | (cg & 1), lane, v);
    const int i = wr * 32 + 16 * qh + li;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = colsub(u, g, a.f32);
      Wl[i][j] = (i < w && j < wc) ? v[u] : 0.0;
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = tid + 256 * q, i = e & 63, j = e >> 6;
      Wl[i][j] = (i < w && j < wc) ? a.C[i + (jc + j) * a.ldc] : 0.0;
    }
  }
  // Tl[k][i] = T[k][i]: the transposed operand of the product
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int e = tid + 256 * q;
    Tl[e & 63][e >> 6] = tv[q];
  }
  __syncthreads();
  const int wave = tid >> 6;
  v4d acc = v4d{0, 0, 0, 0};
#pragma unroll
  for (int k0 = 0; k0 < kLeaf; k0 += 16)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + 4 * g + s;
      acc = mfma(Wl[k][li], Tl[k][16 * wave + li], acc);
    }
  const int i = 16 * wave + li;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int j = 4 * r + g;
    if (i < w && j < wc) out[i + (jc + j) * ldo] = acc[r];
  }
}

void launch_tn_reduce_tmul(const TnArgs& a, const double* T, int w, double* out, int64_t ldo, hipStream_t st,
                           const int* fb, const double* P, int64_t ldp) {
  if (a.M <= 0 || a.N <= 0) return;
  TnArgs b = a;
  // Four workgroups a tile, one batch of 16 loads after the other: the many
  // splits of a tall matrix's few tiles (110: 83 us, 288: 105) are summed by more
  // workgroups first, in place of the coefficients (20 us in all).  Beside the
  // panel chain the second launch costs more than it gains up to some 72 splits
  // (16384 x 2048: 9.57 ms, 9.94 with it).
  if (!a.seq && a.nsplit > 96) {
    b.C = out; b.ldc = ldo; b.C2 = nullptr;
    launch_tn_sum(b, st);
    b.nsplit = 1;
  }
  hipLaunchKernelGGL(tn_reduce_tmul_kernel, dim3(b.ntiles * 4), dim3(256), 0, st, b, T, w, out, ldo, fb, P, ldp);
}

// acc = T^T X with T (64 x 64, upper triangular, row-major LDS): wave v forms
// rows 16v..16v+15, acc[y][r] = (T^T X)[16v + li][16y + 4r + g].  (T^T)[i][k] =
// T[k][i] vanishes for k > i.  X(k, j): X's entries, of which the first NB
// 16-row and 16-column blocks count.
template <int NB, class FX>
__device__ __forceinline__ void tmul(int tid, const double (*Tl)[kLeaf + 1], v4d (&acc)[NB], FX X) {
  const int wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
#pragma unroll
  for (int y = 0; y < NB; ++y) acc[y] = v4d{0, 0, 0, 0};
  if (wave >= NB) return;
#pragma unroll 1
  for (int c = 0; c <= wave; ++c) {
    double xb[4][NB];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int y = 0; y < NB; ++y) xb[s][y] = X(16 * c + 4 * g + s, 16 * y + li);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double xa = Tl[16 * c + 4 * g + s][16 * wave + li];
#pragma unroll
      for (int y = 0; y < NB; ++y) acc[y] = mfma(xb[s][y], xa, acc[y]);
    }
  }
}

// Breakdown fallback of the second pass: the column-wise CGS2 product
// out (w x wn, ld ldo) = P^T Qn over mrows rows, one column of Qn per
// workgroup pass (the coefficients of the next panel against the panel the
// fallback orthogonalised).
template <int NT>
__device__ void colwise_product_store(double* P, int64_t ldp, int64_t mrows, int w, const double* Qn,
                                      int64_t ldqn, int wn, double* out, int64_t ldo, ColwiseLds<NT>& L) {
  const int tid = threadIdx.x;
  for (int jn = 0; jn < wn; ++jn) {
    for (int c0 = 0; c0 < w; c0 += kColChunk)
      colwise_dots<NT>(P, ldp, mrows, c0, min(w, c0 + kColChunk), Qn + (int64_t)jn * ldqn, L.s1, nullptr, -1,
                       1.0, L);
    if (tid < w) out[tid + jn * ldo] = L.s1[tid];
    __syncthreads();
  }
}

// The second pass's breakdown fallback, kept out of line so that its loops
// do not add to the registers of the usual path: CGS2 of the panel into Rl,
// the next panel's coefficients Rbar = P^T Q_next when Q_next is given, and
// its update Q_next -= P Rbar, all by this workgroup.  Returns false for a
// zero column (exact rank deficiency).
__device__ __attribute__((noinline)) bool chol_fallback(const PanelArgs& a, double (*Rl)[kLeaf + 1],
                                                        ColwiseLds<256>* L) {
  const bool ok = colwise_panel<256>(a.P, a.ldp, a.mrows, a.w, Rl, *L);
  if (a.Qn) {
    colwise_product_store<256>(a.P, a.ldp, a.mrows, a.w, a.Qn, a.ldp, a.w, a.Rbar, a.ldr, *L);
    for (int jn = 0; jn < a.w; ++jn) {
      if ((int)threadIdx.x < a.w) L->s2[threadIdx.x] = a.Rbar[threadIdx.x + (int64_t)jn * a.ldr];
      __syncthreads();
      for (int64_t r = threadIdx.x; r < a.mrows; r += 256) {
        double x = a.Qn[r + jn * a.ldp];
        for (int c = 0; c < a.w; ++c) x -= a.P[r + c * a.ldp] * L->s2[c];
        a.Qn[r + jn * a.ldp] = x;
      }
      __syncthreads();
    }
  }
  return ok;
}

// W (w x w Gram matrix, ld ldw) into Rl, identity-padded, Tl the identity, dg
// the diagonal; true if some entry is further than 1e-8 from the identity's.
// flag: a word of LDS.  NB: the 16-column blocks that W has.
template <int NB = 4>
__device__ __forceinline__ bool gram_load(int tid, const double* W, int64_t ldw, int w, double (*Rl)[kLeaf + 1],
                                          double (*Tl)[kLeaf + 1], double* dg, int* flag) {
  const int tx = tid & 63, ty = tid >> 6;
  if (tid == 0) *flag = 0;
  double v[4 * NB];
#pragma unroll
  for (int q = 0; q < 4 * NB; ++q) {
    const int k = ty + 4 * q;   // column (outside W: entry (0, 0), not used)
    const bool in = tx < w && k < w;
    v[q] = W[in ? tx + (int64_t)k * ldw : 0];
    v[q] = in ? v[q] : (tx == k ? 1.0 : 0.0);
  }
  __syncthreads();
  bool far = false;
#pragma unroll
  for (int q = 0; q < 4 * NB; ++q) {
    const int k = ty + 4 * q;
    const double id = tx == k ? 1.0 : 0.0;
    Rl[tx][k] = v[q];
    Tl[tx][k] = id;
    if (k == tx) dg[tx] = v[q];
    far |= !(fabs(v[q] - id) <= 1e-8);
  }
  if (far) *flag = 1;
  __syncthreads();
  return *flag != 0;
}

// chol_blocked out of line, so that its registers do not add to those of the
// kernels that call it: they run beside products of 128 registers whose
// workgroups leave 256 a lane when they end, and a kernel that needs more waits
// for a product's whole grid.
// (The LDS arrays go by LDS pointers: by generic ones every access would test
// for null and add 64-bit addresses.)
typedef __attribute__((address_space(3))) double lds_double;
__device__ __attribute__((noinline)) bool chol_exact(int nb, lds_double* Rl, lds_double* Tl, lds_double* dg) {
  bool bad = false;
  chol_blocked(threadIdx.x, nb, (double (*)[kLeaf + 1])(double*)Rl, (double (*)[kLeaf + 1])(double*)Tl, (double*)dg, bad);
  return bad;
}

// First Cholesky-QR pass by one workgroup: R1 <- chol(W), T <- R1^{-1} (both
// left in Rl and Tl).  Breakdown (a pivot at most kCholBreak times its diagonal
// entry): R1 = T = I, so the transform leaves the panel as it is, and info[1]
// tells the second pass.  store: write R1 (and T, if a.T) and info[1].
template <bool INLINE, int NB = 4>
__device__ __forceinline__ void chol_first(const CholArgs& a, double (*Rl)[kLeaf + 1], double (*Tl)[kLeaf + 1],
                                           double* dg, int* flag, bool store) {
  const int tid = threadIdx.x, tx = tid & 63, ty = tid >> 6, w = a.w;
  gram_load<NB>(tid, a.W, a.ldw, w, Rl, Tl, dg, flag);
  __syncthreads();
  if (tid == 0) *flag = 0;
  bool bad = false;
  if (INLINE)
    chol_blocked(tid, (w + 15) / 16, Rl, Tl, dg, bad);      // (barriers inside)
  else
    bad = chol_exact((w + 15) / 16, (lds_double*)&Rl[0][0], (lds_double*)&Tl[0][0], (lds_double*)dg);
  if (bad) *flag = 1;
  __syncthreads();
  const bool broke = *flag != 0;
  if (broke) {
#pragma unroll
    for (int q = 0; q < 4 * NB; ++q) {
      const int k = ty + 4 * q;
      Rl[tx][k] = Tl[tx][k] = (tx == k) ? 1.0 : 0.0;
    }
    __syncthreads();
  }
  if (!store) return;
#pragma unroll
  for (int q = 0; q < 4 * NB; ++q) {
    const int k = ty + 4 * q;
    if (tx < w && k < w) {
      if (a.T) a.T[tx + k * w] = Tl[tx][k];
      a.R1[tx + k * w] = Rl[tx][k];
    }
  }
  if (tid == 0) a.info[1] = broke;
}

// First pass's transform, and the second pass's Gram product from the same
// rows: a workgroup walks strips of 16 rows of the panel; each strip of
// P (- the split partials of the re-projection update) is multiplied by
// T = R1^{-1} on MFMA, stored to P (and X), and at once multiplied into
// P1^T [P1 | Q_next], whose 64 x 64 blocks stay in registers until the
// workgroup's last strip and are left as split partials (tile 0: Gram, tile 1:
// Q_next) for tn_reduce_split_kernel.  The panel is thus read once for both,
// and the Gram product has no launch of its own.  CHOL: the workgroup runs the
// first pass's Cholesky itself (each of them the same: cheaper than a launch
// of one workgroup before this one); otherwise T comes from memory (the
// factorization ran beside the split update, nn_chol_kernel).
// (gpart == nullptr: the transform alone, for the modes that form the Gram
// product by itself.)
// Latency-bound: 16-row strips let a short panel fill many workgroups.  NB: the
// 16-column blocks that the panel's columns fill (the others are left out: 1386
// x 16 with CHOL 9.3 us, 16.0 with all four; x 35 19.3, 28.8);
// FULL: w = 64, no column masks; NEXT: with Q_next.
template <bool CHOL, int NB, bool FULL, bool NEXT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void panel_first_kernel(PanelArgs a) {
  __builtin_amdgcn_s_setprio(2);   // panel chain
  __shared__ double sT[kLeaf][kLeaf + 1];
  // R1 while it is formed, then the strip before and after its transform and
  // Q_next's rows of it.  (At most 72 KB in all: what a workgroup of the update
  // that runs beside leaves when it ends.)
  __shared__ double sR[CHOL ? kLeaf : (NEXT ? 32 : 16)][kLeaf + 1];
  double (*sP)[kLeaf + 1] = sR, (*sQ)[kLeaf + 1] = sR + 16;
  __shared__ double dg[kLeaf];
  __shared__ int flag;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int w = FULL ? kLeaf : a.w;
  const int strips = (int)((a.mrows + 15) / 16);
  // element u of this thread: row li of the strip, column 16 wave + 4 u + g
  double pv[4], qv[4] = {0.0, 0.0, 0.0, 0.0};
  // (rows and columns outside the panel read row or column 0 and count as zero)
  auto load = [&](int s) {
    const int64_t i = (int64_t)s * 16 + li, ic = i < a.mrows ? i : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = 16 * wave + 4 * u + g;
      const int64_t o = ic + (j < w ? j : 0) * a.ldp;
      pv[u] = a.P[o];
      if (NEXT) qv[u] = a.Qn[o];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool ok = i < a.mrows && 16 * wave + 4 * u + g < w;
      pv[u] = ok ? pv[u] : 0.0;
      qv[u] = NEXT && ok ? qv[u] : 0.0;
    }
  };
  if ((int)blockIdx.x < strips) load(blockIdx.x);
  if constexpr (CHOL) {
    chol_first<false, NB>(a.c, sR, sT, dg, &flag, blockIdx.x == 0);
    __syncthreads();
  } else {
    double tv[4 * NB];
#pragma unroll
    for (int q = 0; q < 4 * NB; ++q) {
      const int e = tid + 256 * q, k = e & 63, j = e >> 6;
      tv[q] = (k < w && j < w) ? a.T[k + j * w] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4 * NB; ++q) {
      const int e = tid + 256 * q;
      sT[e & 63][e >> 6] = tv[q];
    }
  }
  const int ia0 = (wave & 1) * 32, jb0 = (wave >> 1) * 32;     // quadrant of the Gram blocks
  v4d gg[2][2], gq[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) gg[x][y] = gq[x][y] = v4d{0, 0, 0, 0};
  for (int s = blockIdx.x; s < strips; s += gridDim.x) {
    if (a.nsplit > 1) {
      double v[4];
      sum_partials4<8>(a.part, a.nsplit, a.ntiles, s >> 2, s & 3, wave, lane, v);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = 16 * wave + 4 * u + g;
        pv[u] = j < w && (int64_t)s * 16 + li < a.mrows ? pv[u] - v[u] : 0.0;
      }
    }
    __syncthreads();          // T is staged; the previous strip's reads are done
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      sP[li][16 * wave + 4 * u + g] = pv[u];
      if (NEXT) sQ[li][16 * wave + 4 * u + g] = qv[u];
    }
    __syncthreads();
    if (s + (int)gridDim.x < strips) load(s + gridDim.x);
    __builtin_amdgcn_sched_barrier(0);
    v4d acc = v4d{0, 0, 0, 0};
#pragma unroll
    for (int k0 = 0; k0 < 16 * NB; k0 += 16) {
      if (wave >= NB) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = k0 + 4 * g + e;
        acc = mfma(sT[k][16 * wave + li], sP[li][k], acc);
      }
    }
    __syncthreads();
    const int64_t i = (int64_t)s * 16 + li;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = 16 * wave + 4 * r + g;
      sP[li][j] = acc[r];
      if (i < a.mrows && j < w) {
        a.P[i + j * a.ldp] = acc[r];
        if (a.X) a.X[i + j * a.ldx] = acc[r];
      }
    }
    if (!a.gpart) continue;
    __syncthreads();
    if (ia0 >= 16 * NB || jb0 >= 16 * NB) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = 4 * g + e;
      double xa[2], xb[2], xq[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        xa[t] = sP[k][ia0 + 16 * t + li];
        xb[t] = sP[k][jb0 + 16 * t + li];
        xq[t] = NEXT ? sQ[k][jb0 + 16 * t + li] : 0.0;
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          if (ia0 + 16 * x >= 16 * NB || jb0 + 16 * y >= 16 * NB) continue;
          gg[x][y] = mfma(xb[y], xa[x], gg[x][y]);
          if (NEXT) gq[x][y] = mfma(xq[y], xa[x], gq[x][y]);
        }
    }
  }
  if (!a.gpart) return;
  const int tiles = NEXT ? 2 : 1;
  double* mine = a.gpart + part_off(blockIdx.x, tiles, 0, wave) + lane;
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int q = (x * 2 + y) * 4 + r;
        mine[q * 64] = gg[x][y][r];
        if (NEXT) mine[4096 + q * 64] = gq[x][y][r];
      }
}

// Second Cholesky-QR pass from its Gram matrix G = P1^T P1 (and G_next = P1^T
// Q_next): P <- P1 T with T = R2^{-1}, and Q_next -= P Rbar with Rbar = T^T
// G_next, 64 rows at a time.  Every workgroup forms T itself: after a first
// pass W = I + E with |E| <= 1e-8, so R2 = I + F (F the strict upper part of E
// plus half its diagonal) and T = I - F up to O(|E|^2), below rounding; where
// E is larger, the exact factorization runs, in each workgroup the same.  That
// costs less than a launch of one workgroup that the transform has to wait for.
// The last workgroup takes no rows: it stores R_panel = R2 R1 and the copy of T
// for the early update.
// Breakdown (flagged by the first pass, or a pivot here): the last workgroup
// orthogonalises the panel column by column with CGS2 and updates Q_next, the
// others leave it alone; R_panel = R_cgs2 R1, the panel is marked in a.fb for
// the update that started from its first pass, and info[2] counts it.  Only a
// panel that is exactly rank-deficient (a zero column after projection) sets
// info[0].
// NB: the 16-column blocks that the panel's columns fill (the others are left
// out: 1386 x 16 with Q_next 6.8 us, 17.0 with all four; x 35 12.9, 17.7), FULL:
// w = 64 (15.4).
template <int NB, bool FULL, bool NEXT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void panel_second_kernel(PanelArgs a) {
  __builtin_amdgcn_s_setprio(2);   // panel chain
  __shared__ double sT[kLeaf][kLeaf + 1];
  __shared__ double sB[kLeaf][kLeaf + 1];   // W and R2, then Rbar
  __shared__ double dg[kLeaf];
  __shared__ int flag, flag2;
  __shared__ ColwiseLds<256> L;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int w = FULL ? kLeaf : a.w;
  const int tx = lane, ty = wave;
  const bool last = blockIdx.x + 1 == gridDim.x;
  const int tiles = (int)((a.mrows + 63) / 64);
  // rows i = 64 tile + 16 wave + li: columns 16 y + 4 r + g of Q_next; of P,
  // the operand of product m: column 4 m + g, what the accumulators of the
  // transform hold for m = 4 y + r (NEXT), or 16 (m / 4) + 4 g + m % 4
  // (outside the panel: row or column 0, meeting zeros of T, or not stored)
  double xa[4 * NB], cv[4 * NB];
  auto col = [&](int m) { return NEXT ? 4 * m + g : 16 * (m >> 2) + 4 * g + (m & 3); };
  auto load = [&](double (&v)[4 * NB], const double* M, int tile) {
    const int64_t i = (int64_t)tile * 64 + 16 * wave + li, ic = i < a.mrows ? i : 0;
#pragma unroll
    for (int m = 0; m < 4 * NB; ++m) {
      const int j = col(m);
      v[m] = M[ic + (j < w ? j : 0) * a.ldp];
    }
  };
  auto mask = [&](double (&v)[4 * NB]) {
    if (!FULL) {
#pragma unroll
      for (int m = 0; m < 4 * NB; ++m) v[m] = col(m) < w ? v[m] : 0.0;
    }
  };
  double xr[4 * NB];      // Gn; in the last workgroup R1, identity-padded
  if (!last) load(xa, a.P, blockIdx.x);
  if (NEXT || last) {
    const double* M = last ? a.c.R1 : a.Gn;
#pragma unroll
    for (int q = 0; q < 4 * NB; ++q) {
      const int k = ty + 4 * q;
      const bool in = tx < w && k < w;
      xr[q] = M[in ? tx + k * w : 0];
      xr[q] = in ? xr[q] : last && tx == k ? 1.0 : 0.0;
    }
  }
  const bool broke1 = a.c.info[1] != 0;
  const bool far = gram_load<NB>(tid, a.G, w, w, sB, sT, dg, &flag);
  if (tid == 0) flag2 = 0;
  __syncthreads();
  if (!far) {
    double f[4 * NB];
#pragma unroll
    for (int q = 0; q < 4 * NB; ++q) {
      const int i = ty + 4 * q;
      const double e = sB[i][tx];
      f[q] = (i < tx) ? e : (i == tx ? 0.5 * (e - 1.0) : 0.0);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4 * NB; ++q) {
      const int i = ty + 4 * q;
      const double id = (i == tx) ? 1.0 : 0.0;
      sB[i][tx] = id + f[q];
      sT[i][tx] = id - f[q];
    }
  } else if (!broke1) {
    if (chol_exact(NB, (lds_double*)&sB[0][0], (lds_double*)&sT[0][0], (lds_double*)dg)) flag2 = 1;
  }
  __syncthreads();
  const bool fallback = broke1 || flag2 != 0;
  if (!last) {
    if (fallback) return;
    if (NEXT) {
#pragma unroll
      for (int q = 0; q < 4 * NB; ++q) sB[tx][ty + 4 * q] = xr[q];
      __syncthreads();
      v4d rb[NB];
      tmul(tid, sT, rb, [&](int k, int j) { return sB[k][j]; });
      __syncthreads();
#pragma unroll
      for (int y = 0; y < NB; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * wave + li, j = 16 * y + 4 * r + g;
          sB[i][j] = rb[y][r];
          if (blockIdx.x == 0 && i < w && j < w) a.Rbar[i + (int64_t)j * a.ldr] = rb[y][r];
        }
    }
    __syncthreads();
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x - 1) {
      mask(xa);
      if (NEXT) load(cv, a.Qn, tile);         // used after the products
      __builtin_amdgcn_sched_barrier(0);
      v4d pf[NB], acc[NB];
#pragma unroll
      for (int y = 0; y < NB; ++y) pf[y] = acc[y] = v4d{0, 0, 0, 0};
#pragma unroll
      for (int m = 0; m < 4 * NB; ++m) {
#pragma unroll
        for (int y = 0; y < NB; ++y) pf[y] = mfma(sT[col(m)][16 * y + li], xa[m], pf[y]);
      }
      if (tile + (int)gridDim.x - 1 < tiles) load(xa, a.P, tile + gridDim.x - 1);
      // the accumulators hold P[i][4 m + g] for m = 4 y + r: the operand of the
      // second product, lane for lane
      if (NEXT) {
#pragma unroll
        for (int m = 0; m < 4 * NB; ++m) {
#pragma unroll
          for (int y = 0; y < NB; ++y) acc[y] = mfma(sB[4 * m + g][16 * y + li], pf[m >> 2][m & 3], acc[y]);
        }
      }
      const int64_t i = (int64_t)tile * 64 + 16 * wave + li;
      if (i < a.mrows) {
#pragma unroll
        for (int y = 0; y < NB; ++y)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = 16 * y + 4 * r + g;
            if (FULL || j < w) {
              a.P[i + j * a.ldp] = pf[y][r];
              if (NEXT) a.Qn[i + j * a.ldp] = cv[4 * y + r] - acc[y][r];
            }
          }
      }
    }
    return;
  }
  // the last workgroup: T's copy, R_panel = R2 R1
  bool rank_deficient = false;
  if (fallback) {
    rank_deficient = !chol_fallback(a, sB, &L);
    if (tid == 0) {
      a.c.info[2] += 1;
      if (a.fb) *a.fb = 1;
    }
    __syncthreads();
  } else {
    if (a.Tcopy) {
#pragma unroll
      for (int q = 0; q < 4 * NB; ++q) {
        const int k = ty + 4 * q;
        if (tx < w && k < w) a.Tcopy[tx + k * w] = sT[tx][k];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4 * NB; ++q) sT[tx][ty + 4 * q] = xr[q];
  __syncthreads();
  lds_mm_store(tid, sB, sT, w, a.Rout, a.ldr);
  if (tid == 0 && rank_deficient && a.c.info[0] == 0) a.c.info[0] = 1 + a.c.panel;
}

// Workgroups of the first pass: strips of 16 rows shared evenly by at most 128
// of them (their partial Gram blocks, 64 KB each with Q_next, are written and
// read back), 256 for panels of more than 32768 rows, where the rows' own bytes
// outweigh the partials'.
int panel_first_blocks(int64_t mrows, bool gram) {
  const int64_t strips = (mrows + 15) / 16, cap = mrows > 32768 || !gram ? 256 : 128;
  const int64_t per = (strips + cap - 1) / cap;
  return (int)((strips + per - 1) / per);
}

template <bool CHOL, int NB, bool FULL>
static void launch_panel_first_as(const PanelArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)panel_first_blocks(a.mrows, a.gpart != nullptr));
  if (a.Qn && a.gpart)
    hipLaunchKernelGGL((panel_first_kernel<CHOL, NB, FULL, true>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((panel_first_kernel<CHOL, NB, FULL, false>), grid, dim3(256), 0, st, a);
}

template <bool CHOL>
static void launch_panel_first_w(const PanelArgs& a, hipStream_t st) {
  if (a.w == kLeaf) return launch_panel_first_as<CHOL, 4, true>(a, st);
  switch ((a.w - 1) / 16) {
    case 0: return launch_panel_first_as<CHOL, 1, false>(a, st);
    case 1: return launch_panel_first_as<CHOL, 2, false>(a, st);
    case 2: return launch_panel_first_as<CHOL, 3, false>(a, st);
    default: return launch_panel_first_as<CHOL, 4, false>(a, st);
  }
}

void launch_panel_first(const PanelArgs& a, bool chol, hipStream_t st) {
  if (chol)
    launch_panel_first_w<true>(a, st);
  else
    launch_panel_first_w<false>(a, st);
}

// The Gram partials of launch_panel_first summed into G (ld w; Gn from column
// kLeaf on).
void launch_panel_reduce(const PanelArgs& a, hipStream_t st) {
  TnArgs t{};
  t.M = t.M2 = a.w; t.N = a.Qn ? kLeaf + a.w : a.w;
  t.nsplit = panel_first_blocks(a.mrows, true);
  t.tilesN = t.ntiles = a.Qn ? 2 : 1;
  t.C = a.G; t.ldc = a.w;
  t.part = a.gpart;
  t.prio = 1;
  launch_tn_sum(t, st);
}

template <int NB, bool FULL>
static void launch_panel_second_as(const PanelArgs& a, hipStream_t st) {
  const int64_t tiles = (a.mrows + 63) / 64;
  const int64_t per = (tiles + 254) / 255;
  const dim3 grid((unsigned)((tiles + per - 1) / per + 1));
  if (a.Qn)
    hipLaunchKernelGGL((panel_second_kernel<NB, FULL, true>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((panel_second_kernel<NB, FULL, false>), grid, dim3(256), 0, st, a);
}

void launch_panel_second(const PanelArgs& a, hipStream_t st) {
  if (a.w == kLeaf) return launch_panel_second_as<4, true>(a, st);
  switch ((a.w - 1) / 16) {
    case 0: return launch_panel_second_as<1, false>(a, st);
    case 1: return launch_panel_second_as<2, false>(a, st);
    case 2: return launch_panel_second_as<3, false>(a, st);
    default: return launch_panel_second_as<4, false>(a, st);
  }
}

// A panel leaf orthogonalised column by column (the CGS2, ICGS and MGS panel
// modes) by a grid of workgroups, each owning one slab of rows.  A column
// needs a sum over all rows before every update, so each step of the method is
// one launch: it first reduces the partial sums every workgroup of the previous
// launch left (all workgroups sum them redundantly, in the same fixed order, so
// they take identical decisions), then works on its own slab and leaves its
// partial sums for the next launch.  Kernel boundaries order the steps; nothing
// waits inside a launch.
//
// CGS2 / ICGS, one launch per column.  Step j finishes column j-1 and projects
// column j for the first time, both from sums over the same rows:
//   q_{j-2}   = w'_{j-2} / r, r its norm (summed by the step before);
//   w'_{j-1}  = w_{j-1} - Q a, a = Q^T w_{j-1} (the second projection; CGS2
//               always, ICGS when ||w_{j-1}|| < eta ||p_{j-1}||, the DGKS test);
//   p'_j = w_j = p_j - Q t - w'_{j-1} e, t = Q^T p_j, and e = w'_{j-1}^T p_j /
//               ||w'_{j-1}||^2 from the sums at hand: w'^T p = w^T p - a^T t,
//               ||w'||^2 = ||w||^2 - ||a||^2;
//   partials for step j+1: Q^T w_j, Q^T p_{j+1} (w'_{j-1} among Q's columns, not
//               yet normalised: those two are divided by its r there), ||w_j||^2,
//               w_j^T p_{j+1}, ||p_{j+1}||^2, ||w'_{j-1}||^2.
// e enters only the first projection.  Where the second projection changed
// w_{j-1} by more than half (||a||^2 > ||w||^2 / 2, a column nearly dependent on
// its panel) e's relative accuracy is poor, and ICGS takes column j's second
// projection whatever its test says.
// MGS (the paper's sequential MGS), step i: q_{i-1} = u_{i-1} / r; u_c -=
// r_{i-1,c} q_{i-1} for c >= i; partials of ||u_i||^2 and of u_i^T u_c for c > i.
//
// Bound by latency: w + 2 dependent launches a leaf.  A workgroup takes 64 rows
// (more row blocks beyond kColGridMax workgroups); its wave q holds columns
// 16 q .. 16 q + 15 of them, a row per lane, so that the four waves share a
// row's work and the code stays short (the launches' time is largely that of
// fetching it); a wave's sums over its rows end in one transposing butterfly per
// 16 inner products and go straight to memory.  (Two launches per column with 64
// columns a thread took 10 us each: the n = 2048 factorization with ICGS panels
// 48.3 ms, now 23.4: about 7 us a launch and 3 between dependent ones.)
// Partial sums: slots [0, 64) and [64, 128) inner products, 128 .. 131 the others.
constexpr int kColThreads = 256;
enum : int { kSlotT = 64, kSlotW = 128, kSlotU = 129, kSlotP = 130, kSlotN = 131 };
static_assert(kSlotN < kColSlots, "slots");

// r from a squared norm; a zero or non-finite norm flags the panel as exactly
// rank-deficient and leaves the column unnormalised
__device__ __forceinline__ double col_diag(const ColArgs& a, double r2, bool lead) {
  if (!(r2 > 0.0) || !isfinite(r2)) {
    if (lead && a.info[0] == 0) a.info[0] = 1 + a.panel;
    r2 = 1.0;
  }
  return sqrt(r2);
}

// sum over the wavefront
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// red[0 .. kColSlots) = the previous launch's partial sums over G = 32, 64 or 128
// workgroups, in a fixed order, 16 or 32 loads of a thread in flight: two threads
// for each of the first 128 slots, a wave for each of the four others.
__device__ __forceinline__ void col_reduce(const double* in, int G, double* red, double* half) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), slot = tid & 127, h = wave >> 1;
  const double* y = in + 128 + wave + lane * kColSlots;
  const double y0 = y[lane < G ? 0 : -lane * kColSlots], y1 = G > 64 ? y[64 * kColSlots] : 0.0;
  const double* p = in + h * (G / 2) * kColSlots + slot;
  double acc = 0.0;
  auto batch = [&](auto n) {
    constexpr int kN = decltype(n)::value;
    double t[kN];
#pragma unroll
    for (int k = 0; k < kN; ++k) t[k] = p[k * kColSlots];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kN; ++k) acc += t[k];
    p += kN * kColSlots;
  };
  if (G == 32) {
    batch(std::integral_constant<int, 16>{});
  } else {
    for (int g = 0; g < G / 2; g += 32) batch(std::integral_constant<int, 32>{});
  }
  if (h) half[slot] = acc;
  const double n = wave_sum((lane < G ? y0 : 0.0) + y1);
  if (lane == 0) red[128 + wave] = n;
  __syncthreads();
  if (!h) red[slot] = acc + half[slot];
  __syncthreads();
}

// Row r (a valid one) of the wave's 16 columns from c0 on, of which the first
// `cols` are used and the others zero.  All or none are loaded, through one
// advancing address.
__device__ __forceinline__ void col_load(double (&v)[16], const double* P, int64_t ld, int64_t r, int c0, int cols,
                                         int w) {
  if (cols <= 0) {
#pragma unroll
    for (int c = 0; c < 16; ++c) v[c] = 0.0;
    return;
  }
  const double* p = P + r + c0 * ld;
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    v[c] = *p;
    p += c0 + c + 1 < w ? ld : 0;
  }
#pragma unroll
  for (int c = 0; c < 16; ++c) v[c] = c < cols ? v[c] : 0.0;
}

// CGS2 / ICGS step j (0 <= j <= w + 1)
__global__ __launch_bounds__(kColThreads) void colstep_kernel(ColArgs a, int G, int64_t rb, int j, int par) {
  __builtin_amdgcn_s_setprio(2);   // panel chain
  __shared__ double red[kColSlots], half[128];
  // per column: coefficients of the two projections, scale (1, or 1 / r of the
  // column that is not yet normalised)
  __shared__ double ca[kLeaf], ct[kLeaf], cs[kLeaf];
  __shared__ double sums[2][4][64];
  __shared__ double s_aa, s_at;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = blockIdx.x;
  const int w = a.w, c0 = 16 * wave;
  const int64_t ld = a.ldp;
  double* const P = a.P;
  const int64_t r0 = (int64_t)g * rb, r1 = min(a.mrows, r0 + rb);
  const int64_t bufsz = (int64_t)kColGridMax * kColSlots;
  double* out = a.work + par * bufsz + (int64_t)g * kColSlots;
  const double* st_in = a.work + 2 * bufsz + 4 * (par ^ 1);   // [0] ||p_{j-1}||^2, [1] e of the step before, [2] force
  double* st_out = a.work + 2 * bufsz + 4 * par;
  const bool lead = g == 0 && tid == 0;
  const int nq = j < 2 ? 0 : j - 1;       // finished columns; the last of them not yet normalised
  const bool haw = j >= 1 && j <= w, hap = j < w, han = j + 1 < w;    // w_{j-1}, p_j, p_{j+1} exist
  const int kn = nq - 1 - c0, kw = j - 1 - c0;     // columns nq - 1 and j - 1 in the wave's registers (if 0 .. 15)

  double e = 0.0;
  bool second = false;
  double acca[16], acct[16], sw = 0.0, su = 0.0, sp = 0.0, sn = 0.0;
#pragma unroll
  for (int c = 0; c < 16; ++c) acca[c] = acct[c] = 0.0;
  for (int64_t rr = r0; rr < r1; rr += 64) {
    // (rows past the last count as zero)
    const int64_t row = min(rr + lane, r1 - 1);
    const bool act = rr + lane < r1;
    double v[16];
    col_load(v, P, ld, row, c0, nq - c0, w);
    double xw = haw ? P[row + (j - 1) * ld] : 0.0, xp = hap ? P[row + j * ld] : 0.0;
    double xn = han ? P[row + (j + 1) * ld] : 0.0;
    if (rr == r0) {
      // the first block's loads are under way: the reduction of the previous
      // launch's sums, this step's coefficients and column j-1 of R
      double n0 = 0.0, e_prev = 0.0, force = 0.0, inv = 1.0, r = 1.0;
      if (j >= 1) {
        n0 = st_in[0];
        e_prev = st_in[1];
        force = st_in[2];
        col_reduce(a.work + (par ^ 1) * bufsz, G, red, half);
      }
      if (j >= 2) {
        r = col_diag(a, red[kSlotN], lead);
        inv = 1.0 / r;
      }
      const double n1 = red[kSlotW];
      second = haw && j >= 2 && (a.mode == COLWISE_CGS2 || force != 0.0 || n1 < a.eta * a.eta * n0);
      if (wave == 0) {
        // (slots from nq on hold nothing)
        const double s = lane == nq - 1 ? inv : 1.0;
        const double ai = second && lane < nq ? red[lane] * s : 0.0, ti = hap && lane < nq ? red[kSlotT + lane] * s : 0.0;
        ca[lane] = ai;
        ct[lane] = ti;
        cs[lane] = s;
        const double aa = wave_sum(ai * ai), at = wave_sum(ai * ti);
        if (lane == 0) {
          s_aa = aa;
          s_at = at;
        }
        if (g == 0 && lane < nq) {
          double* Rc = a.Rout + (int64_t)(j - 1) * a.ldr + lane;
          if (haw) *Rc = (lane == nq - 1 ? e_prev * r : *Rc) + ai;   // first projection (the step before's), second
          if (hap) Rc[a.ldr] = ti;
          if (lane == nq - 1) Rc[-a.ldr] = r;                        // (row and column j - 2)
        }
      }
      __syncthreads();
      const bool both = haw && hap;
      const double w2 = n1 - s_aa;
      e = both && !(w2 <= 0.0) ? (red[kSlotU] - s_at) / w2 : 0.0;
      if (lead) {
        st_out[0] = j >= 1 ? red[kSlotP] : 0.0;      // ||p_j||^2 before its first projection
        st_out[1] = e;
        st_out[2] = both && second && !(s_aa <= 0.5 * n1) ? 1.0 : 0.0;
      }
    }
    if (!act) {
#pragma unroll
      for (int c = 0; c < 16; ++c) v[c] = 0.0;
      xw = xp = xn = 0.0;
    }
    double s = 0.0, t = 0.0, qn = 0.0;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      v[c] *= cs[c0 + c];
      qn = c == kn ? v[c] : qn;
      s += v[c] * ca[c0 + c];
      t += v[c] * ct[c0 + c];
    }
    if (rr > r0) __syncthreads();   // the block before is done with the sums
    sums[0][wave][lane] = s;
    sums[1][wave][lane] = t;
    __syncthreads();                // (and every wave has read the columns stored below)
    s = sums[0][0][lane] + sums[0][1][lane] + sums[0][2][lane] + sums[0][3][lane];
    t = sums[1][0][lane] + sums[1][1][lane] + sums[1][2][lane] + sums[1][3][lane];
    const double wf = xw - s, pf = xp - t - wf * e;
    if (act) {
      if (kn >= 0 && kn < 16) P[row + (nq - 1) * ld] = qn;
      if (wave == 0) {
        if (second) P[row + (j - 1) * ld] = wf;
        if (hap && j >= 1) P[row + j * ld] = pf;
      }
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const double x = c == kw ? wf : v[c];
      acca[c] += x * pf;
      acct[c] += x * xn;
    }
    sw += pf * pf;
    su += pf * xn;
    sp += xn * xn;
    sn += wf * wf;
  }
  // this workgroup's partial sums
  if (hap && kw >= 0) {
    const double x = colwise_wave_sum16(acca), y = colwise_wave_sum16(acct);
    if (lane < 16) {
      out[c0 + lane] = x;
      out[kSlotT + c0 + lane] = y;
    }
  }
  const double x = wave_sum(wave == 0 ? sw : wave == 1 ? su : wave == 2 ? sp : sn);
  if (lane == 0) out[kSlotW + wave] = x;
  // after the last step: zeros below R's diagonal
  if (j == w + 1 && g == 0)
    for (int q = tid; q < w * w; q += kColThreads)
      if (q % w > q / w) a.Rout[q % w + (int64_t)(q / w) * a.ldr] = 0.0;
}

// MGS step i (0 <= i <= w)
__global__ __launch_bounds__(kColThreads) void colmgs_kernel(ColArgs a, int G, int64_t rb, int i, int par) {
  __builtin_amdgcn_s_setprio(2);   // panel chain
  __shared__ double red[kColSlots], half[128];
  __shared__ double coef[kLeaf];          // r_{i-1,c} of the columns c in [i, w), zero elsewhere
  __shared__ double su[2][64];            // u_i of the row block
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = blockIdx.x;
  const int w = a.w, c0 = 16 * wave;
  const int64_t ld = a.ldp;
  double* const P = a.P;
  const int64_t r0 = (int64_t)g * rb, r1 = min(a.mrows, r0 + rb);
  const int64_t bufsz = (int64_t)kColGridMax * kColSlots;
  double* out = a.work + par * bufsz + (int64_t)g * kColSlots;
  const bool lead = g == 0 && tid == 0;
  const bool mine = c0 + 16 > i;          // some of the wave's columns are still to be orthogonalised
  const int ki = i - c0;                  // column i in the wave's registers (if 0 .. 15)
  double inv = 1.0;
  double acc[16], sn = 0.0;
#pragma unroll
  for (int c = 0; c < 16; ++c) acc[c] = 0.0;
  for (int64_t rr = r0; rr < r1; rr += 64) {
    const int64_t row = min(rr + lane, r1 - 1);
    const bool act = rr + lane < r1;
    double v[16];
    col_load(v, P, ld, row, c0, mine ? w - c0 : 0, w);
    double xq = i > 0 ? P[row + (i - 1) * ld] : 0.0;
    if (rr == r0 && i > 0) {
      col_reduce(a.work + (par ^ 1) * bufsz, G, red, half);
      const double r = col_diag(a, red[kSlotW], lead);
      inv = 1.0 / r;
      if (lead) a.Rout[(i - 1) + (int64_t)(i - 1) * a.ldr] = r;
      if (tid < kLeaf) coef[tid] = tid >= i && tid < w ? red[tid] * inv : 0.0;
      if (g == 0 && tid >= i && tid < w) a.Rout[(i - 1) + (int64_t)tid * a.ldr] = red[tid] * inv;
    }
    if (!act) {
#pragma unroll
      for (int c = 0; c < 16; ++c) v[c] = 0.0;
      xq = 0.0;
    }
    __syncthreads();                // the coefficients; every wave has read column i - 1
    if (i > 0) {
      const double q = xq * inv;
      if (act && wave == 0) P[row + (i - 1) * ld] = q;
      if (mine) {
        double* p = P + row + c0 * ld;
#pragma unroll
        for (int c = 0; c < 16; ++c, p += ld) {
          v[c] -= coef[c0 + c] * q;
          if (act && c >= ki && c0 + c < w) *p = v[c];
        }
      }
    }
    if (i < w) {
      double u = 0.0;
#pragma unroll
      for (int c = 0; c < 16; ++c) u = c == ki ? v[c] : u;
      const int buf = (rr - r0) >> 6 & 1;
      if (ki >= 0 && ki < 16) su[buf][lane] = u;
      __syncthreads();
      u = su[buf][lane];
#pragma unroll
      for (int c = 0; c < 16; ++c) acc[c] += v[c] * u;
      sn += u * u;
    }
  }
  if (i < w) {
    if (mine) {
      const double x = colwise_wave_sum16(acc);
      if (lane < 16) out[c0 + lane] = x;
    }
    if (wave == 0) {
      const double n = wave_sum(sn);
      if (lane == 0) out[kSlotW] = n;
    }
  } else if (g == 0) {
    for (int q = tid; q < w * w; q += kColThreads)
      if (q % w > q / w) a.Rout[q % w + (int64_t)(q / w) * a.ldr] = 0.0;
  }
}

// The launches of one leaf: w + 2 for CGS2 / ICGS, w + 1 for MGS; whole row
// blocks of 64 shared evenly by 32 or 64 workgroups (128 from 16384 rows on:
// their sums are read by every workgroup of the next launch).  Workgroups left
// without rows leave zeros.
void launch_colpanel(const ColArgs& a, hipStream_t st) {
  const int64_t blocks = (a.mrows + 63) / 64;
  const int G = blocks <= 32 ? 32 : blocks <= 256 ? 64 : kColGridMax;
  const int64_t per = (blocks + G - 1) / G;
  int par = 0;
  const bool mgs = a.mode == COLWISE_MGS;
  for (int j = 0; j <= (mgs ? a.w : a.w + 1); ++j, par ^= 1)
    if (mgs)
      hipLaunchKernelGGL(colmgs_kernel, dim3(G), dim3(kColThreads), 0, st, a, G, 64 * per, j, par);
    else
      hipLaunchKernelGGL(colstep_kernel, dim3(G), dim3(kColThreads), 0, st, a, G, 64 * per, j, par);
}

CholArgs chol_args(const double* W, int64_t ldw, int w, int panel, const Scratch& s) {
  CholArgs c{};
  c.W = W; c.ldw = ldw;
  c.w = w; c.panel = panel;
  c.T = s.T; c.R1 = s.R1; c.info = s.info;
  return c;
}

// --------------------------------------------------------------------------
// Rank-K update  C -= A B  (A: M x K, B: K x N, C: M x N, column-major).
// Tile 64 x 64 per block; wave w takes rows 16w..16w+15 and all 64 columns
// (4 accumulator blocks).  K advances in slabs of 64: the B slab (64 x 64) is
// staged in LDS and shared by the four waves, each lane keeps its 16 A values
// of a slab in registers, and the next slab's A and B loads are in flight
// while the current slab is multiplied (two A register sets alternate
// explicitly).  Short K (the trailing update, K = b): C is loaded at the start
// so all of a tile's loads are in flight together.  Long K with few tiles
// (re-projection): the K range is split over blocks and nn_reduce_kernel
// subtracts the partial tiles from C in split order.
// --------------------------------------------------------------------------

constexpr int NK = 64;   // k per slab of the rank-K update
// Fewest columns for which the update takes the 128 x 128 kernel.
constexpr int kQuadMinN = 256;

// Shared pieces of the rank-K update kernels.  B staging: thread t moves
// B[k0 + 16(t & 3) + e][jb + (t >> 2)], e < 16 (8 vector loads from one
// column); columns past N read column 0 and feed only unstored outputs.
struct NnTile {
  int tm, tn, wave, lane, li, g, tid;
  int64_t i, ic;
  int jb;
  bool aok;
  const double* ar;   // A[ic][g]: lane (li, g) supplies A[i][k0 + 4m + g] to product m
  const double* bp;   // B[16(t & 3)][jb + (t >> 2)]
};

__device__ __forceinline__ NnTile nn_tile_at(const NnArgs& a, int tm, int tn) {
  NnTile t;
  t.tm = tm;
  t.tn = tn;
  t.tid = threadIdx.x;
  t.wave = t.tid >> 6;
  t.lane = t.tid & 63;
  t.li = t.lane & 15;
  t.g = t.lane >> 4;
  t.i = (int64_t)t.tm * 64 + t.wave * 16 + t.li;
  t.jb = t.tn * 64;
  t.aok = t.i < a.M;
  t.ic = t.aok ? t.i : 0;            // clamped row: valid address, result unused
  t.ar = a.A + t.ic + (int64_t)t.g * a.lda;
  const int jc = t.jb + (t.tid >> 2);
  t.bp = a.B + 16 * (t.tid & 3) + (int64_t)(jc < a.N ? jc : 0) * a.ldb;
  return t;
}

// XCD-aware tile order for one-pass updates.  Workgroups are dealt to the
// eight XCDs round-robin (block b runs on XCD b mod 8), and each XCD has its
// own L2.  Block b takes position start(x) + b / 8 of an order in which the
// tiles come in four bands of row tiles, each band walked column slab by
// column slab; XCD x's positions form one contiguous range of that order,
// i.e. about half of one band.  Each XCD thus reads a quarter of the A rows
// and half of the B columns instead of all of both.
__device__ __forceinline__ void xcd_tile(int b, int ntiles, int tilesM, int tilesN, int& tm, int& tn) {
  const int x = b & 7, j = b >> 3;
  const int q = ntiles >> 3, r = ntiles & 7;
  const int pos = x * q + (x < r ? x : r) + j;
  const int bm = (tilesM + 3) >> 2;                 // row tiles per band
  const int band = pos / (bm * tilesN);
  const int rows = min(bm, tilesM - band * bm);     // rows in this band (the last may be short)
  const int in = pos - band * bm * tilesN;
  tn = in / rows;
  tm = band * bm + in % rows;
}

__device__ __forceinline__ void nn_load_a(const NnArgs& a, const NnTile& t, int k0, double (&xa)[16]) {
#pragma unroll
  for (int m = 0; m < 16; ++m) xa[m] = t.ar[(int64_t)(k0 + 4 * m) * a.lda];
}

__device__ __forceinline__ void nn_load_b(const NnTile& t, int k0, v2d (&rb)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) rb[e] = *reinterpret_cast<const v2d*>(t.bp + k0 + 2 * e);
}

__device__ __forceinline__ void nn_put_b(double (*sBb)[64 + 1], const NnTile& t, const v2d (&rb)[8]) {
  const int kq = 16 * (t.tid & 3), j = t.tid >> 2;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    sBb[kq + 2 * e][j] = rb[e].x;
    sBb[kq + 2 * e + 1][j] = rb[e].y;
  }
}

// Partial slab [k0, ke): zero beyond ke on both operands (scalar loads).
__device__ __forceinline__ void nn_load_tail(const NnArgs& a, const NnTile& t, int k0, int ke, double (&xa)[16],
                                             double (*sBb)[64 + 1]) {
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const int k = k0 + 4 * m + t.g;
    xa[m] = (k < ke) ? t.ar[(int64_t)(k0 + 4 * m) * a.lda] : 0.0;
  }
  const int kq = 16 * (t.tid & 3), j = t.tid >> 2;
#pragma unroll
  for (int e = 0; e < 16; ++e) sBb[kq + e][j] = (k0 + kq + e < ke) ? t.bp[k0 + e] : 0.0;
}

template <class Acc>
__device__ __forceinline__ void nn_mma(Acc (&acc)[4], const double (*sBb)[64 + 1], const NnTile& t,
                                       const double (&xa)[16]) {
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const int k = 4 * m + t.g;
#pragma unroll
    for (int y = 0; y < 4; ++y) acc[y] = mfma(sBb[k][16 * y + t.li], xa[m], acc[y]);
  }
}

// C -= A B for K <= 64 (K < 64, or operands nnw_kernel does not take):
// every load of the tile (C, A, the B slab) is issued before the first
// product.  The tile loop is
// grid-strided; launched with one block per tile it runs once.  This form
// compiles to more registers than the straight-line one (three waves per SIMD
// instead of four), and measured faster in the factorization: the update's
// blocks leave more room for the panel chain's kernels that run beside them.
template <int TAG>
__global__ __launch_bounds__(256) void nn1_kernel(NnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  typedef v4d Acc;
  __shared__ double sB[NK][64 + 1];
  for (int blk = blockIdx.x; blk < a.ntiles; blk += gridDim.x) {
    int tm, tn;
    xcd_tile(blk, a.ntiles, a.ntiles / a.tilesN, a.tilesN, tm, tn);
    const NnTile t = nn_tile_at(a, tm, tn);
    double cval[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = t.jb + 16 * (e >> 2) + colsub(e & 3, t.g, false);
      cval[e] = a.C[t.ic + (int64_t)(j < a.N ? j : 0) * a.ldc];
    }
    double xa[16];
    if (blk != (int)blockIdx.x) __syncthreads();   // the previous tile's reads of sB are done
    if (a.K == NK && a.vec) {
      v2d rb[8];
      nn_load_a(a, t, 0, xa);
      nn_load_b(t, 0, rb);
      __builtin_amdgcn_sched_barrier(0);
      nn_put_b(sB, t, rb);
    } else {
      nn_load_tail(a, t, 0, a.K, xa, sB);
    }
    __syncthreads();
    Acc acc[4];
#pragma unroll
    for (int y = 0; y < 4; ++y) acc[y] = Acc{0, 0, 0, 0};
    nn_mma(acc, sB, t, xa);
    if (t.aok) {
#pragma unroll
      for (int y = 0; y < 4; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = t.jb + 16 * y + colsub(r, t.g, false);
          if (j < a.N) a.C[t.i + (int64_t)j * a.ldc] = cval[y * 4 + r] - acc[y][r];
        }
    }
  }
}

// Long K: slabs of 64 with the next slab's A and B loads in flight while the
// current slab is multiplied (A register sets alternate explicitly).  SPLIT:
// the block's K range is one split and its partial tile is stored for
// nn_reduce_kernel; otherwise C is updated in place (the path for operands
// nnw_kernel does not take), FLUSH: after every slab.
template <bool SPLIT, int TAG, bool FLUSH = false>
__device__ __forceinline__ void nn_body(const NnArgs& a, double (*sB)[NK][64 + 1], int bx, int split) {
  typedef v4d Acc;
  int tm = bx / a.tilesN, tn = bx % a.tilesN;
  if (!SPLIT) xcd_tile(bx, a.ntiles, a.ntiles / a.tilesN, a.tilesN, tm, tn);
  const NnTile t = nn_tile_at(a, tm, tn);
  const int kb = split * a.kchunk;
  const int ke = std::min(a.K, kb + a.kchunk);
  const int nfull = a.vec ? (ke - kb) / NK : 0;
  // in-place update: C's loads go out before the products, so their latency
  // overlaps the K loop instead of following it
  double cval[16];
  if (!SPLIT) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = t.jb + 16 * (e >> 2) + colsub(e & 3, t.g, false);
      cval[e] = a.C[t.ic + (int64_t)(j < a.N ? j : 0) * a.ldc];
    }
  }
  Acc acc[4];
#pragma unroll
  for (int y = 0; y < 4; ++y) acc[y] = Acc{0, 0, 0, 0};
  auto flush = [&]() {
    if constexpr (!FLUSH) return;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      cval[e] -= acc[e >> 2][e & 3];
      acc[e >> 2][e & 3] = 0.0;
    }
  };
  auto koff = [&](int sl) { return kb + std::min(sl, nfull - 1) * NK; };
  if (nfull > 0) {
    double xa0[16], xa1[16];
    v2d rb[8];
    nn_load_a(a, t, koff(0), xa0);
    nn_load_b(t, koff(0), rb);
    __builtin_amdgcn_sched_barrier(0);
    nn_put_b(sB[0], t, rb);
    __syncthreads();
    int sl = 0;
    for (; sl + 2 <= nfull; sl += 2) {
      nn_load_a(a, t, koff(sl + 1), xa1);
      nn_load_b(t, koff(sl + 1), rb);
      __builtin_amdgcn_sched_barrier(0);
      nn_mma(acc, sB[0], t, xa0);
      flush();
      __builtin_amdgcn_sched_barrier(0);
      nn_put_b(sB[1], t, rb);
      __syncthreads();
      nn_load_a(a, t, koff(sl + 2), xa0);
      nn_load_b(t, koff(sl + 2), rb);
      __builtin_amdgcn_sched_barrier(0);
      nn_mma(acc, sB[1], t, xa1);
      flush();
      __builtin_amdgcn_sched_barrier(0);
      nn_put_b(sB[0], t, rb);
      __syncthreads();
    }
    if (sl < nfull) {
      nn_mma(acc, sB[0], t, xa0);
      flush();
    }
  }
  const int kt = kb + nfull * NK;
  for (int k0 = kt; k0 < ke; k0 += NK) {
    // partial (or unaligned) slabs; the buffer not read by the last full slab
    const int buf = ((k0 - kb) / NK) & 1;
    double xa[16];
    nn_load_tail(a, t, k0, ke, xa, sB[buf]);
    __syncthreads();
    nn_mma(acc, sB[buf], t, xa);
    flush();
    __syncthreads();
  }
  if (SPLIT) {
    double* mine = a.part + part_off(split, a.ntiles, bx, t.wave);
#pragma unroll
    for (int y = 0; y < 4; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) mine[(y * 4 + r) * 64 + t.lane] = acc[y][r];
    return;
  }
  if (!t.aok) return;
#pragma unroll
  for (int y = 0; y < 4; ++y)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = t.jb + 16 * y + colsub(r, t.g, false);
      if (j < a.N) a.C[t.i + (int64_t)j * a.ldc] = cval[y * 4 + r] - acc[y][r];
    }
}

template <bool SPLIT, int TAG, bool FLUSH = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void nn_kernel(NnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ double sB[2][NK][64 + 1];
  nn_body<SPLIT, TAG, FLUSH>(a, sB, blockIdx.x, blockIdx.y);
}

// The same update where 64 x 64 tiles would leave the chip idle, as tns_kernel
// does for the product: a workgroup forms 16 x 16 elements of C, its 4 waves
// share the depth, 16 k-values at a time in turn, straight from memory, and
// their sums are added through LDS in order.  No partials, so the split
// update's second launch (or its sum in panel_first) goes too.
constexpr int kSmallNnWaves = 4;

__device__ __forceinline__ void nns_body(const NnArgs& a, double (*red)[4][64], int bx) {
  const int tilesM = (int)((a.M + 15) / 16);
  const int64_t i0 = (int64_t)(bx % tilesM) * 16;
  const int j0 = bx / tilesM * 16;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // rows and columns outside the matrix read row and column 0 and are not stored
  const int64_t i = i0 + li, ic = i < a.M ? i : 0;
  const int j = j0 + 4 * wave + g;
  double* pc = a.C + ic + (int64_t)(j < a.N ? j : 0) * a.ldc;
  const double old = *pc;
  const double* pa = a.A + ic + 4 * g * a.lda;
  const double* pb = a.B + 4 * g + (int64_t)(j0 + li < a.N ? j0 + li : 0) * a.ldb;
  const int nfull = a.K / 16;
  const int mine = (nfull - wave + kSmallNnWaves - 1) / kSmallNnWaves;      // the wave's whole chunks
  v4d acc = v4d{0, 0, 0, 0};
  double x0[8], x1[8], y0[8], y1[8];
  auto load = [&](double (&x)[8], int q) {
    const int k = 16 * (wave + q * kSmallNnWaves);
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = pa[(int64_t)(k + s) * a.lda];
    if (a.vec) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const v2d v = *reinterpret_cast<const v2d*>(pb + k + 2 * h);
        x[4 + 2 * h] = v.x; x[5 + 2 * h] = v.y;
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) x[4 + s] = pb[k + s];
    }
  };
  auto mac = [&](const double (&x)[8]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = mfma(x[4 + s], x[s], acc);
  };
  if (mine > 0) load(x0, 0);
  if (mine > 1) load(x1, 1);
#pragma unroll 1
  for (int q = 0; q < mine; q += 4) {
    if (q + 2 < mine) load(y0, q + 2);
    if (q + 3 < mine) load(y1, q + 3);
    mac(x0);
    if (q + 1 < mine) mac(x1);
    if (q + 4 < mine) load(x0, q + 4);
    if (q + 5 < mine) load(x1, q + 5);
    if (q + 2 < mine) mac(y0);
    if (q + 3 < mine) mac(y1);
  }
  if (const int k0 = 16 * nfull; k0 < a.K && wave == nfull % kSmallNnWaves) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool in = k0 + 4 * g + s < a.K;
      x0[s] = in ? pa[(int64_t)(k0 + s) * a.lda] : 0.0;
      x0[4 + s] = in ? pb[k0 + s] : 0.0;
    }
    mac(x0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][r][lane] = acc[r];
  __syncthreads();
  double v = 0.0;
#pragma unroll
  for (int e = 0; e < kSmallNnWaves; ++e) v += red[e][wave][lane];     // element r = wave of the accumulators
  if (i < a.M && j < a.N) *pc = old - v;
}

template <int TAG>
__global__ __launch_bounds__(64 * kSmallNnWaves) void nns_kernel(NnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ double red[kSmallNnWaves][4][64];
  nns_body(a, red, blockIdx.x);
}

// The re-projection update P -= Q S, split over K, with one extra block that
// runs the panel's first Cholesky-QR pass: the factorization reads only the
// Gram rows of the preceding product and the update only its coefficient
// rows, so the single-block Cholesky runs alongside the update's blocks
// instead of after them on the panel chain.  Block column x = ntiles holds the
// Cholesky (its y > 0 blocks exit at once); both uses share the LDS layout
// size (two 64 x 65 double arrays).  SMALL: the update by nns_body, unsplit,
// with the Cholesky in the first block.
template <bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void nn_chol_kernel(NnArgs a,
                                                                                               CholArgs c) {
  __builtin_amdgcn_s_setprio(2);
  __shared__ double smem[2 * NK * (64 + 1)];
  __shared__ double dg[kLeaf];
  __shared__ int flag;
  if ((int)blockIdx.x == (SMALL ? 0 : a.ntiles)) {
    if (blockIdx.y == 0)
      chol_first<true>(c, reinterpret_cast<double (*)[kLeaf + 1]>(smem),
                 reinterpret_cast<double (*)[kLeaf + 1]>(smem + kLeaf * (kLeaf + 1)), dg, &flag, true);
    return;
  }
  if constexpr (SMALL)
    nns_body(a, reinterpret_cast<double (*)[4][64]>(smem), blockIdx.x - 1);
  else
    nn_body<true, TAG_REPROJ>(a, reinterpret_cast<double (*)[NK][64 + 1]>(smem), blockIdx.x, blockIdx.y);
}

// C -= sum of the split partials (split order).  One block per wave of a
// tile, thread (qg, lane) owns the lane's 4 values of column block qg.
__global__ __launch_bounds__(256) void nn_reduce_kernel(NnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  const int tile = blockIdx.x >> 2, wave = blockIdx.x & 3;
  const int tm = tile / a.tilesN, tn = tile % a.tilesN;
  const int qg = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int64_t i = (int64_t)tm * 64 + wave * 16 + li;
  const int jq = tn * 64 + 16 * qg;            // + colsub(u, g)
  const bool aok = i < a.M;
  const int64_t ic = aok ? i : 0;
  double old[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = jq + colsub(u, g, false);
    old[u] = a.C[ic + (int64_t)(j < a.N ? j : 0) * a.ldc];
  }
  double v[4];
  sum_partials4(a.part, a.nsplit, a.ntiles, tile, wave, qg, lane, v);
  if (!aok) return;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = jq + colsub(u, g, false);
    if (j < a.N) a.C[i + (int64_t)j * a.ldc] = old[u] - v[u];
  }
}

NnArgs nn_setup(double* C, int64_t ldc, const double* A, int64_t lda, const double* B, int64_t ldb, int64_t M,
                int N, int K, const Scratch& s) {
  NnArgs a{};
  a.C = C; a.ldc = ldc; a.A = A; a.lda = lda; a.B = B; a.ldb = ldb;
  a.M = M; a.N = N; a.K = K;
  a.tilesN = (N + 63) / 64;
  a.ntiles = (int)((M + 63) / 64) * a.tilesN;
  a.part = s.part;
  a.vec = aligned16(B, ldb);
  // few tiles and a long reduction: split K so at most 512 blocks (two per
  // CU, one wave of blocks) run, each over at least 2 slabs
  int ns = 1;
  if (K > NK && a.ntiles < 512 && K >= 4 * NK) {
    ns = (int)std::min<int64_t>(std::max(1, 512 / a.ntiles), K / (2 * NK));
    while (ns > 1 && (int64_t)ns * a.ntiles > s.npart) --ns;
  }
  int kchunk = (K + ns - 1) / ns;
  kchunk = (kchunk + NK - 1) / NK * NK;
  ns = (K + kchunk - 1) / kchunk;
  a.kchunk = kchunk;
  a.nsplit = ns;
  return a;
}

// Tile and k range [klo, khi) of workgroup b in the adjoint's products, whose
// operands may be triangular; false for a tile that is not needed.  The XCDs
// take workgroups in turn and the tiles' work is uneven, so they are dealt with
// the row index fastest (every XCD gets each column's rows in equal shares,
// long columns first; xcd_tile's contiguous ranges would give some XCDs twice
// the work of others), rotated by the column where rows differ too.
__device__ __forceinline__ bool nn_tri_tile(const NnArgs& a, int b, int tilesM, int T, int& tm, int& tn, int& klo,
                                            int& khi) {
  tn = b / tilesM;
  tm = b - tn * tilesM;
  if (a.tri & TRI_C_LOWER) {
    tm += tn;
    if (tm >= tilesM) return false;
  }
  const int i0 = tm * T, j0 = tn * T;
  if (a.tri & TRI_A_UPPER) klo = i0;
  if ((a.tri & TRI_B_LOWER) && j0 > klo) klo = j0;
  if ((a.tri & TRI_B_UPPER) && j0 + T < khi) khi = j0 + T;
  return true;
}

// In-place rank-K update C (M x N) -= A (M x K) B (K x N) for K >= 64 (the
// trailing update, long unsplit re-projections), with
// the product kernel's pipeline: 64 x 64 output tile per block, 4 waves each
// a 32 x 32 quadrant, both operands staged through LDS in slabs of KC
// k-values (slab s multiplied while slab s+1 lands in one register set and
// slab s+2 is requested into the other).  A (i contiguous) is transposed into
// the product kernel's [i][k] LDS layout as it is staged; B (k contiguous)
// is staged as there.  C's loads are issued before the K loop.  Requires K a
// multiple of KC, 16-byte aligned A and B with even leading dimensions, and
// an even M; tiles take the XCD-aware order.
// The body for slabs of SK k-values (32 or 16; LDS row pitch SK + 2).
// FLUSH: the accumulators are subtracted from C's elements and cleared after
// every a.flush k-values (a multiple of 32).
template <int TAG, int SK, bool FLUSH = false>
__device__ __forceinline__ void nnw_body(const NnArgs& a, double (*sA)[64 * (SK + 2)], double (*sB)[64 * (SK + 2)]) {
  typedef v4d Acc;
  constexpr int LW = SK + 2;         // padded LDS row (doubles)
  constexpr int NQ = SK / 8;         // v2d loads per thread and operand per slab
  constexpr int TPC = SK / 2;        // B staging: threads per column (one k pair each)
  constexpr int CPP = 256 / TPC;     // B staging: columns per pass
  int tm, tn;
  int klo = 0, khi = a.K;
  if constexpr (TAG == TAG_ADJ) {
    if (!nn_tri_tile(a, blockIdx.x, a.ntiles / a.tilesN, 64, tm, tn, klo, khi)) return;
  } else {
    xcd_tile(blockIdx.x, a.ntiles, a.ntiles / a.tilesN, a.tilesN, tm, tn);
  }
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int ia0 = (wave & 1) * 32, jb0 = (wave >> 1) * 32;
  const int64_t ib = (int64_t)tm * 64, jb = (int64_t)tn * 64;
  // C's 16 values of this lane (quadrant element (x, y, r)); rows and
  // columns outside C read row or column 0 and are not stored
  double cval[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int x = e >> 3, y = (e >> 2) & 1, r = e & 3;
    const int64_t i = ib + ia0 + 16 * x + li, j = jb + jb0 + 16 * y + colsub(r, g, false);
    if constexpr (TAG == TAG_ADJ)
      cval[e] = a.Cin ? a.Cin[(i < a.M ? i : 0) + (j < a.N ? j : 0) * a.ldcin] : 0.0;
    else
      cval[e] = a.C[(i < a.M ? i : 0) + (j < a.N ? j : 0) * a.ldc];
  }
  // staging of A: thread loads one v2d (rows 2 ip, 2 ip + 1) of k rows kr + 8 q
  const int ip = tid & 31, kr = tid >> 5;
  const int64_t ia = ib + 2 * ip;
  const double* ga = a.A + (ia + 1 < a.M ? ia : 0) + (int64_t)(klo + kr) * a.lda;
  // staging of B: thread loads one v2d (k pair lq) of columns lc + CPP q
  const int lc = tid / TPC, lq = tid % TPC;
  const double* gb[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int64_t j = jb + lc + CPP * q;
    gb[q] = a.B + klo + (j < a.N ? j : 0) * a.ldb + 2 * lq;
  }
  Acc acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = Acc{0, 0, 0, 0};
  const int nsl = (khi - klo) / SK;
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < SK; kk += 16) {
      double xa[2][4], xb[2][4];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const double* pa = &sA[buf][(ia0 + 16 * t + li) * LW + kk + 4 * g];
        const double* pb = &sB[buf][(jb0 + 16 * t + li) * LW + kk + 4 * g];
        v2d a0 = *reinterpret_cast<const v2d*>(pa), a1 = *reinterpret_cast<const v2d*>(pa + 2);
        v2d b0 = *reinterpret_cast<const v2d*>(pb), b1 = *reinterpret_cast<const v2d*>(pb + 2);
        xa[t][0] = a0.x; xa[t][1] = a0.y; xa[t][2] = a1.x; xa[t][3] = a1.y;
        xb[t][0] = b0.x; xb[t][1] = b0.y; xb[t][2] = b1.x; xb[t][3] = b1.y;
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) acc[x][y] = mfma(xb[y][s], xa[x][s], acc[x][y]);
    }
  };
  // slab sl's first k (clamped to the last slab: prefetches past the end
  // reload cached data that is never used)
  auto koff = [&](int sl) { return (int64_t)std::min(sl, nsl - 1) * SK; };
  v2d ra0[NQ], rb0[NQ], ra1[NQ], rb1[NQ];
  auto load = [&](v2d (&ra)[NQ], v2d (&rb)[NQ], int64_t k) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      ra[q] = *reinterpret_cast<const v2d*>(ga + (k + 8 * q) * a.lda);
      rb[q] = *reinterpret_cast<const v2d*>(gb[q] + k);
    }
  };
  auto put = [&](int buf, const v2d (&ra)[NQ], const v2d (&rb)[NQ]) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      sA[buf][(2 * ip) * LW + kr + 8 * q] = ra[q].x;
      sA[buf][(2 * ip + 1) * LW + kr + 8 * q] = ra[q].y;
      *reinterpret_cast<v2d*>(&sB[buf][(lc + CPP * q) * LW + 2 * lq]) = rb[q];
    }
  };
  load(ra0, rb0, koff(0));
  load(ra1, rb1, koff(1));
  put(0, ra0, rb0);
  __syncthreads();
  int sl = 0;
  for (; sl + 2 <= nsl; sl += 2) {
    load(ra0, rb0, koff(sl + 2));
    __builtin_amdgcn_sched_barrier(0);
    compute(0);
    __builtin_amdgcn_sched_barrier(0);
    put(1, ra1, rb1);
    __syncthreads();
    load(ra1, rb1, koff(sl + 3));
    __builtin_amdgcn_sched_barrier(0);
    compute(1);
    __builtin_amdgcn_sched_barrier(0);
    put(0, ra0, rb0);
    if constexpr (FLUSH)
      if ((sl + 2) * SK % a.flush == 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          cval[e] -= acc[e >> 3][e >> 2 & 1][e & 3];
          acc[e >> 3][e >> 2 & 1][e & 3] = 0.0;
        }
      }
    __syncthreads();
  }
  if (sl < nsl) compute(0);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int x = e >> 3, y = (e >> 2) & 1, r = e & 3;
    const int64_t i = ib + ia0 + 16 * x + li, j = jb + jb0 + 16 * y + colsub(r, g, false);
    double v = acc[x][y][r];
    if constexpr (TAG == TAG_ADJ) v *= a.sign;
    if (i < a.M && j < a.N) a.C[i + j * a.ldc] = cval[e] - v;
  }
}

// 32-deep slabs, two waves per SIMD: the rank-64 trailing update, which runs
// beside the panel chain (with 16-deep slabs and three waves per SIMD it is
// faster alone but the step at n = 4096 was 3.8% slower).
template <int TAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void nnw_kernel(NnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ double sA[2][64 * (32 + 2)];
  __shared__ double sB[2][64 * (32 + 2)];
  nnw_body<TAG, 32>(a, sA, sB);
}

// 16-deep slabs (37 KB of LDS, 148-164 VGPRs), three waves per SIMD: K >= 128,
// where the update is MFMA-bound in FP64.  Against the 32-deep form, 9% faster
// alone at K = 128 and 8% at K = 256, and 4% off the n = 16384 step.
// FLUSH: updates whose sums may not be as deep as K.  C's elements are in
// registers already, so it costs one subtraction per element and flush (n = 4096,
// K = 128 with a flush at 64, against nnq_kernel without: the step takes 13.0 ms
// instead of 12.7, with panels updated one by one 13.3).
template <int TAG, bool FLUSH = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void nnw16_kernel(NnArgs a) {
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ double sA[2][64 * (16 + 2)];
  __shared__ double sB[2][64 * (16 + 2)];
  nnw_body<TAG, 16, FLUSH>(a, sA, sB);
}

// 128 x 128 output tile per workgroup (512 threads, 2 x 4 waves, each wave
// 64 rows x 32 columns), 16-deep slabs double-buffered in LDS (72 KB) with
// one register set of staged loads, two workgroups per CU: K >= 128.  Each
// staged column of A and row of B feeds 128 outputs instead of 64, which
// halves the L2 requests per flop against nnw16_kernel.  Alone, the
// K = 256 update of a 49152 x 32768 C runs at 58.7 TFLOP/s against 51.3
// (K = 128, 32768 x 20480: 48.1 against 41.1).  A (i contiguous) is
// transposed into the [i][k] LDS layout as it is staged; C is read after
// the K loop, one 16-row block at a time, and written back in place.
// Requires K a multiple of 16, 16-byte aligned A and B with even leading
// dimensions, and an even M; tiles take the XCD-aware order.
template <int TAG>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void nnq_kernel(NnArgs a) {
  constexpr int SK = 16, LW = SK + 2;
  constexpr int AKR = 8;               // A staging: k rows per pass (64 row pairs x 8)
  constexpr int TPC = SK / 2, CPP = 512 / TPC;   // B staging: 8 threads per column, 64 columns a pass
  if (a.prio) __builtin_amdgcn_s_setprio(2);
  __shared__ double sA[2][128 * LW];
  __shared__ double sB[2][128 * LW];
  const int tilesM = (int)((a.M + 127) / 128), tilesN = (a.N + 127) / 128;
  int tm, tn;
  int klo = 0, khi = a.K;
  if constexpr (TAG == TAG_ADJ) {
    if (!nn_tri_tile(a, blockIdx.x, tilesM, 128, tm, tn, klo, khi)) return;
  } else {
    xcd_tile(blockIdx.x, tilesM * tilesN, tilesM, tilesN, tm, tn);
  }
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int ia0 = 64 * (wave & 1), jb0 = 32 * (wave >> 1);
  const int64_t ib = (int64_t)tm * 128, jb = (int64_t)tn * 128;
  const int ip = tid & 63, kr = tid >> 6;
  const int64_t ia = ib + 2 * ip;
  const double* ga = a.A + (ia + 1 < a.M ? ia : 0) + (int64_t)(klo + kr) * a.lda;
  const int lc = tid / TPC, lq = tid % TPC;
  const double* gb[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int64_t j = jb + lc + CPP * q;
    gb[q] = a.B + klo + (j < a.N ? j : 0) * a.ldb + 2 * lq;
  }
  v4d acc[4][2];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = v4d{0, 0, 0, 0};
  auto compute = [&](int buf) {
#pragma unroll
    for (int s0 = 0; s0 < 4; s0 += 2) {
      double xa[4][2], xb[2][2];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const v2d v = *reinterpret_cast<const v2d*>(&sA[buf][(ia0 + 16 * t + li) * LW + 4 * g + s0]);
        xa[t][0] = v.x; xa[t][1] = v.y;
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const v2d v = *reinterpret_cast<const v2d*>(&sB[buf][(jb0 + 16 * t + li) * LW + 4 * g + s0]);
        xb[t][0] = v.x; xb[t][1] = v.y;
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) acc[x][y] = mfma(xb[y][s], xa[x][s], acc[x][y]);
    }
  };
  const int nsl = (khi - klo) / SK;
  v2d ra[2], rb[2];
  auto load = [&](int64_t k) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      ra[q] = *reinterpret_cast<const v2d*>(ga + (k + AKR * q) * a.lda);
      rb[q] = *reinterpret_cast<const v2d*>(gb[q] + k);
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      sA[buf][(2 * ip) * LW + kr + AKR * q] = ra[q].x;
      sA[buf][(2 * ip + 1) * LW + kr + AKR * q] = ra[q].y;
      *reinterpret_cast<v2d*>(&sB[buf][(lc + CPP * q) * LW + 2 * lq]) = rb[q];
    }
  };
  load(0);
  put(0);
  __syncthreads();
  for (int sl = 0; sl < nsl; ++sl) {
    if (sl + 1 < nsl) load((int64_t)(sl + 1) * SK);
    __builtin_amdgcn_sched_barrier(0);
    compute(sl & 1);
    __builtin_amdgcn_sched_barrier(0);
    if (sl + 1 < nsl) put((sl + 1) & 1);
    __syncthreads();
  }
  // C -= acc, one 16-row block of the wave's 64 rows at a time; rows and
  // columns outside C read row or column 0 and are not stored
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int64_t i = ib + ia0 + 16 * x + li;
    double cv[2][4];
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t j = jb + jb0 + 16 * y + colsub(r, g, false);
        if constexpr (TAG == TAG_ADJ)
          cv[y][r] = a.Cin ? a.Cin[(i < a.M ? i : 0) + (j < a.N ? j : 0) * a.ldcin] : 0.0;
        else
          cv[y][r] = a.C[(i < a.M ? i : 0) + (j < a.N ? j : 0) * a.ldc];
      }
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t j = jb + jb0 + 16 * y + colsub(r, g, false);
        double v = acc[x][y][r];
        if constexpr (TAG == TAG_ADJ) v *= a.sign;
        if (i < a.M && j < a.N) a.C[i + j * a.ldc] = cv[y][r] - v;
      }
  }
}

static unsigned nns_grid(const NnArgs& a) { return (unsigned)((a.M + 15) / 16 * ((a.N + 15) / 16)); }

// Up to 1280 workgroups (2048 of one slab) the 64 x 64 tiles lose to these (us;
// 5120 x 64 x 320: 20.4 and 11.1; x 768: 26.1 and 22.9; 2304 x 256 x 64: 6.6
// and 6.5), beyond a depth of 1024, where each workgroup's reads count, fewer
// (1386 x 35 x 1386, 258 of them: 18.8 and 17.6; x 64, 344: 18.9 and 19.7).
bool nn_small(NnArgs& a) {
  const int64_t wgs = nns_grid(a);
  if (a.K > 1024 ? wgs * a.K > 400000 : wgs > (a.K <= NK ? 2048 : 1280)) return false;
  a.small = 1;
  a.nsplit = 1;
  return true;
}

// Operands the LDS-staged update takes, K >= 64 (else the register-staged
// kernels): 18-22% faster standalone than the register-staged long-K kernel
// at K = 128 and 256.  At K = 64 it is ~8% slower alone than nn1_kernel but
// 1% faster in the factorization, beside the panel chain's kernels.
static bool nnw_ok(const NnArgs& a) {
  return a.K >= NK && a.K % KC == 0 && a.M % 2 == 0 && aligned16(a.A, a.lda) && aligned16(a.B, a.ldb);
}

// The 128 x 128 update: K >= 128 and at least two 128-wide tiles each way
// (see kQuadMinN for the column count).
static bool nnq_ok(const NnArgs& a) {
  return nnw_ok(a) && a.K >= 2 * NK && a.M >= 256 && a.N >= kQuadMinN;
}

// nnw16_kernel's slabs come in pairs of 16 k-values, nn_kernel's are of 64 (it
// subtracts after each); both hold C beside the sums, for which nnq_kernel has no
// registers.
void nn_flush(NnArgs& a, int depth) {
  a.flush = nnw_ok(a) && depth % KC == 0 ? depth : NK;
  a.nsplit = 1;
}

template <int TAG>
static void nn_launch_tag(const NnArgs& a, hipStream_t st) {
  if (a.flush && nnw_ok(a))
    hipLaunchKernelGGL((nnw16_kernel<TAG, true>), dim3(a.ntiles), dim3(256), 0, st, a);
  else if (a.flush)
    hipLaunchKernelGGL((nn_kernel<false, TAG, true>), dim3(a.ntiles), dim3(256), 0, st, a);
  else if (a.small)
    hipLaunchKernelGGL((nns_kernel<TAG>), dim3(nns_grid(a)), dim3(64 * kSmallNnWaves), 0, st, a);
  else if (a.K <= NK && !nnw_ok(a))
    hipLaunchKernelGGL((nn1_kernel<TAG>), dim3(a.ntiles), dim3(256), 0, st, a);
  else if (a.nsplit > 1)
    hipLaunchKernelGGL((nn_kernel<true, TAG>), dim3(a.ntiles, a.nsplit), dim3(256), 0, st, a);
  else if (nnq_ok(a))
    hipLaunchKernelGGL((nnq_kernel<TAG>), dim3((unsigned)(((a.M + 127) / 128) * ((a.N + 127) / 128))), dim3(512), 0,
                       st, a);
  else if (nnw_ok(a) && a.K >= 2 * NK)
    hipLaunchKernelGGL((nnw16_kernel<TAG>), dim3(a.ntiles), dim3(256), 0, st, a);
  else if (nnw_ok(a))
    hipLaunchKernelGGL((nnw_kernel<TAG>), dim3(a.ntiles), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((nn_kernel<false, TAG>), dim3(a.ntiles, 1), dim3(256), 0, st, a);
}

void launch_nn_product(const NnArgs& a, int tag, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return;
  switch (tag) {
    case TAG_TRAIL: nn_launch_tag<TAG_TRAIL>(a, st); break;
    case TAG_REPROJ: nn_launch_tag<TAG_REPROJ>(a, st); break;
    default: nn_launch_tag<TAG_PANEL>(a, st); break;
  }
}

// The adjoint's products: C = Cin - sign A B with C, Cin apart and triangular
// operands' zero tiles left out.  The kernel by size as in nn_launch_tag;
// false, launching nothing, for operands the LDS-staged kernels do not take.
bool launch_nn_adj(const NnArgs& a, hipStream_t st) {
  if (!nnw_ok(a)) return false;
  // (fewer 128 x 128 blocks than the chip holds leave it idle: 64 x 64 tiles then)
  const int64_t blocks = ((a.M + 127) / 128) * ((a.N + 127) / 128);
  if (nnq_ok(a) && blocks >= 512)
    hipLaunchKernelGGL((nnq_kernel<TAG_ADJ>), dim3((unsigned)blocks), dim3(512), 0, st, a);
  else
    hipLaunchKernelGGL((nnw16_kernel<TAG_ADJ>), dim3(a.ntiles), dim3(256), 0, st, a);
  return true;
}

bool launch_nn_chol(const NnArgs& a, const CholArgs& c, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0 || c.w > kLeaf) return false;
  if (a.small) {
    hipLaunchKernelGGL((nn_chol_kernel<true>), dim3(nns_grid(a) + 1), dim3(256), 0, st, a, c);
    return true;
  }
  if (a.K <= NK || a.nsplit <= 1) return false;
  hipLaunchKernelGGL((nn_chol_kernel<false>), dim3(a.ntiles + 1, a.nsplit), dim3(256), 0, st, a, c);
  return true;
}

void launch_nn_reduce(const NnArgs& a, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0 || a.K <= NK || a.nsplit <= 1) return;
  hipLaunchKernelGGL(nn_reduce_kernel, dim3(a.ntiles * 4), dim3(256), 0, st, a);
}

}  // namespace cqr
