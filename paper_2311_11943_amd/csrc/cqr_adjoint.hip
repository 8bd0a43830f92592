// Memory-bound kernels of the adjoint (reverse-mode derivative) of the coded
// QR and of the coded solve.  The dense products of the adjoint (Q~^T dQ~,
// R dR^T, Q~ copyltu(M), D R^{-T}) run on the MFMA product kernels; these
// kernels transpose, symmetrize, form outer products and matrix-vector
// products, and fold the checksum rows back onto A.
#include "cqr_kernels.hpp"
#include "cqr_mfma.hpp"

namespace cqr {

constexpr int kAdjThreads = 256;

static unsigned blocks_for(int64_t n) {
  int64_t b = (n + kAdjThreads - 1) / kAdjThreads;
  return (unsigned)(b < 1 ? 1 : b);
}

// dst (cols x rows) = scale * src^T (src rows x cols), through a 64 x 64 LDS
// tile so both the loads and the stores cover contiguous columns.  upper:
// entries of src below its diagonal are taken as zero.
__global__ __launch_bounds__(kAdjThreads) void transpose_kernel(const double* src, int64_t lds, double* dst,
                                                                int64_t ldd, int64_t rows, int64_t cols, double scale,
                                                                int upper) {
  __shared__ double t[64][65];
  const int64_t i0 = (int64_t)blockIdx.x * 64, j0 = (int64_t)blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int c = ty; c < 64; c += 4) {
    const int64_t i = i0 + tx, j = j0 + c;
    double v = 0.0;
    if (i < rows && j < cols && (!upper || i <= j)) v = src[i + j * lds];
    t[tx][c] = v;
  }
  __syncthreads();
  for (int c = ty; c < 64; c += 4) {
    const int64_t j = j0 + tx, i = i0 + c;
    if (j < cols && i < rows) dst[j + i * ldd] = scale * t[c][tx];
  }
}

// C <- copyltu(C) (n x n): every entry above the diagonal takes the value of
// its mirror below it.  Reads only the lower triangle, writes only the upper.
__global__ __launch_bounds__(kAdjThreads) void copyltu_kernel(double* C, int64_t ldc, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * kAdjThreads + threadIdx.x;
  if (e >= n * n) return;
  const int64_t i = e % n, j = e / n;
  if (i < j) C[i + j * ldc] = C[j + i * ldc];
}

// C[i][j] = scale * sum_{r < k} U[i][r] V[j][r]  (rows x cols; U has rowsu rows,
// zero from there on); with upper, entries below the diagonal are zero.  Bound
// by its stores: a thread owns two rows (256 apart) of kOuterCols columns, its
// U entries read once per right-hand side.
constexpr int kOuterCols = 8;

__global__ __launch_bounds__(kAdjThreads) void outer_kernel(const double* U, int64_t ldu, const double* V,
                                                            int64_t ldv, int64_t rowsu, int64_t rows, int64_t cols,
                                                            int k, double scale, int upper, double* C, int64_t ldc) {
  const int64_t i0 = (int64_t)blockIdx.x * (2 * kAdjThreads) + threadIdx.x, j0 = (int64_t)blockIdx.y * kOuterCols;
  double acc[2][kOuterCols];
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int c = 0; c < kOuterCols; ++c) acc[e][c] = 0.0;
  for (int r = 0; r < k; ++r) {
    double u[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int64_t i = i0 + e * kAdjThreads;
      u[e] = i < rowsu ? U[i + r * ldu] : 0.0;
    }
#pragma unroll
    for (int c = 0; c < kOuterCols; ++c) {
      const double v = j0 + c < cols ? V[j0 + c + r * ldv] : 0.0;
#pragma unroll
      for (int e = 0; e < 2; ++e) acc[e][c] += u[e] * v;
    }
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int64_t i = i0 + e * kAdjThreads;
#pragma unroll
    for (int c = 0; c < kOuterCols; ++c) {
      const int64_t j = j0 + c;
      if (i < rows && j < cols) C[i + j * ldc] = i < rowsu && (!upper || i <= j) ? scale * acc[e][c] : 0.0;
    }
  }
}

// y[i][r] = sum_j A[i][j] x[j][r]  (A m x n, x n x nrhs).  A workgroup takes 64
// rows; its wave q sums a quarter of the columns, eight columns of A in flight
// (a row's whole sum in one thread left a chain of n / 8 round trips to memory),
// and the quarters are added in order.
__global__ __launch_bounds__(kAdjThreads) void gemv_n_kernel(const double* A, int64_t lda, int64_t m, int n,
                                                             const double* x, int64_t ldx, int nrhs, double* y,
                                                             int64_t ldy) {
  __shared__ double part[kAdjThreads / 64][64];
  // (the wave's index made uniform, so x comes through scalar loads)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const double* ai = A + (i < m ? i : 0);
  const int per = (n + kAdjThreads / 64 - 1) / (kAdjThreads / 64);
  const int jb = wave * per, je = jb + per < n ? jb + per : n;
  constexpr int kB = 8;
  for (int r = 0; r < nrhs; ++r) {
    const double* xr = x + (int64_t)r * ldx;
    double acc = 0.0;
    int j = jb;
    for (; j + kB <= je; j += kB) {
      double a[kB];
#pragma unroll
      for (int t = 0; t < kB; ++t) a[t] = ai[(int64_t)(j + t) * lda];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < kB; ++t) acc += a[t] * xr[j + t];
    }
    for (; j < je; ++j) acc += ai[(int64_t)j * lda] * xr[j];
    part[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && i < m) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < kAdjThreads / 64; ++q) s += part[q][lane];
      y[i + (int64_t)r * ldy] = s;
    }
    __syncthreads();
  }
}

// dA = X_top + G_v^T X_bottom:  block t of dA (rows t bs .. t bs + bs) is
// X_t + sum_k g~_v[k][t] X_{p_r + k}.  Thread = (row r in a block, column c);
// the K_v checksum values are read once and reused for every block t.
__global__ __launch_bounds__(kAdjThreads) void fold_kernel(FoldArgs a) {
  const int64_t e = (int64_t)blockIdx.x * kAdjThreads + threadIdx.x;
  if (e >= a.bs * a.cols) return;
  const int64_t r = e % a.bs, c = e / a.bs;
  const double* x = a.X + c * a.ldx + r;
  double* d = a.dA + c * a.ldd + r;
  double chk[kMaxGen];
#pragma unroll
  for (int k = 0; k < kMaxGen; ++k) chk[k] = k < a.kv ? x[a.m + k * a.bs] : 0.0;
  for (int t = 0; t < a.pr; ++t) {
    double v = x[t * a.bs];
#pragma unroll
    for (int k = 0; k < kMaxGen; ++k)
      if (k < a.kv) v += a.gv[k * a.pr + t] * chk[k];
    d[t * a.bs] = v;
  }
}

// Y (n x n) = the block diagonal of the 64 x 64 tiles in T (tile k at
// T + 4096 k, column-major), zeros elsewhere: the inverted diagonal blocks of
// an upper-triangular matrix laid out as the start of its inverse.
__global__ __launch_bounds__(kAdjThreads) void blockdiag_kernel(const double* T, double* Y, int64_t ldy, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * kAdjThreads + threadIdx.x;
  if (e >= n * n) return;
  const int64_t i = e % n, j = e / n;
  Y[i + j * ldy] = (i >> 6) == (j >> 6) ? T[(i >> 6) * 4096 + (i & 63) + (j & 63) * 64] : 0.0;
}

// One product of a doubling level of the triangular inverse, all pairs of
// adjacent h-blocks [i0, i0 + h), [i0 + h, i0 + h + h2) in one launch (grid z):
//   SECOND false:  W = R12 T22     (T22 upper triangular: k <= j)
//   SECOND true:   T12 = -T11 W    (T11 upper triangular: k >= i)
// 64 x 64 output tile per workgroup, 4 waves each a 32 x 32 quadrant, 16-deep
// slabs through LDS, the next slab's loads in flight; any alignment.  Latency
// binds it (few tiles and short depths), so the pairs share a launch: at
// n = 2048 the whole inverse takes 10 launches up to h = 512 instead of 150.
template <bool SECOND>
__global__ __launch_bounds__(256) void inv_level_kernel(const double* R, int64_t ldr, double* Rinv, double* W,
                                                        int64_t n, int64_t h) {
  __shared__ double sA[2][16][64 + 2];      // [k][i]
  __shared__ double sB[2][64][16 + 2];      // [j][k]
  const int64_t i0 = (int64_t)blockIdx.z * 2 * h, c0 = i0 + h;
  const int64_t h2 = n - c0 < h ? n - c0 : h;
  const int64_t ib = (int64_t)blockIdx.x * 64, jb = (int64_t)blockIdx.y * 64;
  if (jb >= h2) return;
  const double* A = SECOND ? Rinv + i0 + i0 * n : R + i0 + c0 * ldr;
  const int64_t lda = SECOND ? n : ldr;
  const double* B = SECOND ? W + i0 + c0 * n : Rinv + c0 + c0 * n;
  double* C = (SECOND ? Rinv : W) + i0 + c0 * n;
  const int64_t klo = SECOND ? ib : 0;
  const int64_t khi = SECOND ? h : (jb + 64 < h2 ? jb + 64 : h2);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int ia0 = (wave & 1) * 32, jb0 = (wave >> 1) * 32;
  const int bk = tid & 15, bj = tid >> 4;
  double ra[4], rb[4];
  auto load = [&](int64_t k0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t k = k0 + wave + 4 * q;
      ra[q] = k < khi ? A[ib + lane + k * lda] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t j = jb + bj + 16 * q;
      rb[q] = k0 + bk < khi && j < h2 ? B[k0 + bk + j * n] : 0.0;
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sA[buf][wave + 4 * q][lane] = ra[q];
      sB[buf][bj + 16 * q][bk] = rb[q];
    }
  };
  v4d acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = v4d{0, 0, 0, 0};
  load(klo);
  put(0);
  __syncthreads();
  int buf = 0;
  for (int64_t k0 = klo; k0 < khi; k0 += 16, buf ^= 1) {
    if (k0 + 16 < khi) load(k0 + 16);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double xa[2], xb[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        xa[t] = sA[buf][4 * g + s][ia0 + 16 * t + li];
        xb[t] = sB[buf][jb0 + 16 * t + li][4 * g + s];
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = mfma(xb[y], xa[x], acc[x][y]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (k0 + 16 < khi) put(buf ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = ib + ia0 + 16 * x + li, j = jb + jb0 + 16 * y + 4 * r + g;
        if (j < h2) C[i + j * n] = SECOND ? -acc[x][y][r] : acc[x][y][r];
      }
}

void launch_inv_level(const double* R, int64_t ldr, double* Rinv, double* W, int64_t n, int64_t h, bool second,
                      hipStream_t st) {
  if (h >= n) return;
  const dim3 grid((unsigned)(h / 64), (unsigned)(h / 64), (unsigned)((n - h + 2 * h - 1) / (2 * h)));
  if (second)
    hipLaunchKernelGGL(inv_level_kernel<true>, grid, dim3(256), 0, st, R, ldr, Rinv, W, n, h);
  else
    hipLaunchKernelGGL(inv_level_kernel<false>, grid, dim3(256), 0, st, R, ldr, Rinv, W, n, h);
}

// C *= s (rows x cols, ld ldc)
__global__ __launch_bounds__(kAdjThreads) void scale_kernel(double* C, int64_t ldc, int64_t rows, int64_t cols,
                                                            double s) {
  const int64_t e = (int64_t)blockIdx.x * kAdjThreads + threadIdx.x;
  if (e >= rows * cols) return;
  C[e % rows + (e / rows) * ldc] *= s;
}

void launch_blockdiag(const double* T, double* Y, int64_t ldy, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(blockdiag_kernel, dim3(blocks_for(n * n)), dim3(kAdjThreads), 0, st, T, Y, ldy, n);
}

void launch_scale(double* C, int64_t ldc, int64_t rows, int64_t cols, double s, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return;
  hipLaunchKernelGGL(scale_kernel, dim3(blocks_for(rows * cols)), dim3(kAdjThreads), 0, st, C, ldc, rows, cols, s);
}

// dst = src (rows x cols)
__global__ __launch_bounds__(kAdjThreads) void copy_kernel(const double* src, int64_t lds, double* dst, int64_t ldd,
                                                           int64_t rows, int64_t cols) {
  const int64_t e = (int64_t)blockIdx.x * kAdjThreads + threadIdx.x;
  if (e >= rows * cols) return;
  dst[e % rows + (e / rows) * ldd] = src[e % rows + (e / rows) * lds];
}

void launch_copy(const double* src, int64_t lds, double* dst, int64_t ldd, int64_t rows, int64_t cols,
                 hipStream_t st) {
  if (rows <= 0 || cols <= 0) return;
  hipLaunchKernelGGL(copy_kernel, dim3(blocks_for(rows * cols)), dim3(kAdjThreads), 0, st, src, lds, dst, ldd, rows,
                     cols);
}

void launch_transpose(const double* src, int64_t lds, double* dst, int64_t ldd, int64_t rows, int64_t cols,
                      double scale, bool upper, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return;
  const dim3 grid((unsigned)((rows + 63) / 64), (unsigned)((cols + 63) / 64));
  hipLaunchKernelGGL(transpose_kernel, grid, dim3(kAdjThreads), 0, st, src, lds, dst, ldd, rows, cols, scale,
                     upper ? 1 : 0);
}

void launch_copyltu(double* C, int64_t ldc, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(copyltu_kernel, dim3(blocks_for(n * n)), dim3(kAdjThreads), 0, st, C, ldc, n);
}

void launch_outer(const double* U, int64_t ldu, const double* V, int64_t ldv, int64_t rowsu, int64_t rows,
                  int64_t cols, int k, double scale, bool upper, double* C, int64_t ldc, hipStream_t st) {
  const dim3 grid((unsigned)((rows + 2 * kAdjThreads - 1) / (2 * kAdjThreads)),
                  (unsigned)((cols + kOuterCols - 1) / kOuterCols));
  hipLaunchKernelGGL(outer_kernel, grid, dim3(kAdjThreads), 0, st, U, ldu, V, ldv, rowsu, rows, cols, k, scale,
                     upper ? 1 : 0, C, ldc);
}

void launch_gemv_n(const double* A, int64_t lda, int64_t m, int n, const double* x, int64_t ldx, int nrhs,
                   double* y, int64_t ldy, hipStream_t st) {
  hipLaunchKernelGGL(gemv_n_kernel, dim3((unsigned)((m + 63) / 64)), dim3(kAdjThreads), 0, st, A, lda, m, n, x, ldx,
                     nrhs, y, ldy);
}

void launch_fold(const FoldArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(fold_kernel, dim3(blocks_for(a.bs * a.cols)), dim3(kAdjThreads), 0, st, a);
}


}  // namespace cqr
