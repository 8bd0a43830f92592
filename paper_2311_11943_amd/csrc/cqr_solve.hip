// Coded linear solve (the linear-solve equations that follow the
// post-orthogonalization theorem):  X = R_1^{-1} (Qpost^T Bpost).
//   1. gemv_t_kernel: Y = Qpost^T Bpost, one wave per column of Qpost (its m
//      entries are contiguous), partial sums reduced across the wave.
//   2. trinv_kernel: every 64 x 64 diagonal block of R_1 is inverted at once
//      (one workgroup per block).
//   3. trsv_flow_kernel: the block back substitution, one launch of dependent
//      workgroups (one per 128 rows and four right-hand sides).
#include "cqr_kernels.hpp"
#include "cqr_mfma.hpp"

#include <mutex>

namespace cqr {

constexpr int kSolveThreads = 256;
constexpr int kSolveBlock = 64;      // diagonal block of the back substitution
constexpr int kRhsChunk = 4;         // right-hand sides per pass
constexpr long long kUnset = -1;     // bit pattern of an entry of X not yet solved (a NaN)

// Y = Q^T B: WPC waves share a column of Q (its m entries are contiguous), a
// wave takes every WPC-th run of 64 rows; their sums are added in order.  Bound
// by reading Q: one wave per column leaves a tall matrix with few columns too
// little in flight (65536 x 512, one right-hand side: 140 us with one wave per
// column, 68 with four).  The rows after the last whole batch are a batch too,
// its loads masked: one after the other they took 1350 us of 1024 rows, 64 columns
// and 1024 right-hand sides, and 530 so (4096 rows, whole batches: 1000).
template <int WPC>
__global__ __launch_bounds__(kSolveThreads) void gemv_t_kernel(const double* Q, int64_t ldq, int64_t m, int n,
                                                               const double* B, int64_t ldb, int nrhs, double* Y,
                                                               int64_t ldy) {
  __shared__ double part[kSolveThreads / 64][kRhsChunk];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = blockIdx.x * (kSolveThreads / 64 / WPC) + wave / WPC, w0 = wave % WPC;
  const double* q = Q + (int64_t)(col < n ? col : 0) * ldq;
  constexpr int kBatch = 8;   // rows per lane whose loads are issued together
  for (int r0 = 0; r0 < nrhs; r0 += kRhsChunk) {
    const int nr = nrhs - r0 < kRhsChunk ? nrhs - r0 : kRhsChunk;
    double acc[kRhsChunk] = {0.0, 0.0, 0.0, 0.0};
    int64_t i = w0 * 64 + lane;
    for (; i + (kBatch - 1) * 64 * WPC < m; i += kBatch * 64 * WPC) {
      double qv[kBatch], bv[kBatch][kRhsChunk];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        qv[j] = q[i + j * 64 * WPC];
#pragma unroll
        for (int t = 0; t < kRhsChunk; ++t)
          bv[j][t] = t < nr ? B[i + j * 64 * WPC + (int64_t)(r0 + t) * ldb] : 0.0;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
#pragma unroll
        for (int t = 0; t < kRhsChunk; ++t) acc[t] += qv[j] * bv[j][t];
    }
    if (i - lane < m) {             // the last rows, as one batch
      double qv[kBatch], bv[kBatch][kRhsChunk];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const int64_t r = i + j * 64 * WPC;
        qv[j] = 0.0;
#pragma unroll
        for (int t = 0; t < kRhsChunk; ++t) bv[j][t] = 0.0;
        if (r >= m) continue;
        qv[j] = q[r];
#pragma unroll
        for (int t = 0; t < kRhsChunk; ++t)
          if (t < nr) bv[j][t] = B[r + (int64_t)(r0 + t) * ldb];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
#pragma unroll
        for (int t = 0; t < kRhsChunk; ++t) acc[t] += qv[j] * bv[j][t];
    }
#pragma unroll
    for (int t = 0; t < kRhsChunk; ++t) {
      double v = acc[t];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      if (WPC == 1) {
        if (lane == 0 && col < n && t < nr) Y[col + (int64_t)(r0 + t) * ldy] = v;
      } else if (lane == 0) {
        part[wave][t] = v;
      }
    }
    if (WPC > 1) {
      __syncthreads();
      if (w0 == 0 && lane < nr && col < n) {
        double v = 0.0;
#pragma unroll
        for (int e = 0; e < WPC; ++e) v += part[wave + e][lane];
        Y[col + (int64_t)(r0 + lane) * ldy] = v;
      }
      __syncthreads();
    }
  }
}

// T_kk = R_kk^{-1} for block k = blockIdx.x (w = min(64, n - 64k) rows; the
// 64 x 64 output is padded with the identity).  T is column-major, 64 x 64 per
// block, zero below the diagonal.  Bound by its serial chain, so the chain is
// kept to 16 pivots: wave q inverts diagonal block q (16 x 16, lane j < 16 back
// substitutes column j of the identity in registers), then block column b = q
// of T follows on MFMA, T_ab = -T_aa sum_{c = a+1..b} R_ac T_cb for a = b-1
// down to 0.  (64 pivots with a barrier each took 115 us at n = 4096; this form
// takes 11.6.)
// X != nullptr (the coded solve): rows 64k .. 64k + w of the nrhs columns of X
// are set to kUnset for trsv_flow_kernel.
__global__ __launch_bounds__(kSolveThreads) void trinv_kernel(const double* R, int64_t ldr, int64_t n, double* T,
                                                              double* X, int64_t ldx, int nrhs) {
  __shared__ double Rl[kSolveBlock][kSolveBlock + 1];
  __shared__ double Tl[kSolveBlock][kSolveBlock + 1];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int64_t k0 = (int64_t)blockIdx.x * kSolveBlock;
  const int w = (int)((n - k0) < kSolveBlock ? (n - k0) : kSolveBlock);
  {
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int c = wave + 4 * q;
      v[q] = (lane < w && c < w && lane <= c) ? R[(k0 + lane) + (k0 + c) * ldr] : (lane == c ? 1.0 : 0.0);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      Rl[lane][wave + 4 * q] = v[q];
      Tl[lane][wave + 4 * q] = 0.0;
    }
  }
  if (X && lane < w)
    for (int r = wave; r < nrhs; r += kSolveThreads / 64)
      X[k0 + lane + (int64_t)r * ldx] = __longlong_as_double(kUnset);
  __syncthreads();
  const int o = 16 * wave;
  if (lane < 16) {
    double s[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = i == lane ? 1.0 : 0.0;
#pragma unroll
    for (int i = 15; i >= 0; --i) {
      s[i] /= Rl[o + i][o + i];
#pragma unroll
      for (int k = 0; k < i; ++k) s[k] -= Rl[o + k][o + i] * s[i];
      Tl[o + i][o + lane] = i <= lane ? s[i] : 0.0;
    }
  }
  __syncthreads();
#pragma unroll 1
  for (int a = wave - 1; a >= 0; --a) {
    v4d acc = v4d{0, 0, 0, 0};
#pragma unroll 1
    for (int c = a + 1; c <= wave; ++c)
      mma16(acc, lane, 1, [&](int i, int k) { return Rl[16 * a + i][16 * c + k]; },
            [&](int k, int j) { return Tl[16 * c + k][o + j]; });
    // staged in T's own block (only this wave touches block column `wave`)
#pragma unroll
    for (int r = 0; r < 4; ++r) Tl[16 * a + li][o + 4 * r + g] = acc[r];
    __builtin_amdgcn_wave_barrier();
    v4d t = v4d{0, 0, 0, 0};
    mma16(t, lane, 1, [&](int i, int k) { return Tl[16 * a + i][16 * a + k]; },
          [&](int k, int j) { return Tl[16 * a + k][o + j]; });
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r) Tl[16 * a + li][o + 4 * r + g] = -t[r];
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  double* out = T + (int64_t)blockIdx.x * kSolveBlock * kSolveBlock;
#pragma unroll
  for (int q = 0; q < 16; ++q) out[lane + (wave + 4 * q) * kSolveBlock] = Tl[lane][wave + 4 * q];
}

// R_1 X = Y (n x nrhs) in one launch, for the dependent chain that bounds it:
// a workgroup takes one block of 128 rows and up to four right-hand sides,
// subtracts R_1[rows, j] x_j for the blocks j below it as their x_j appear, and
// then solves its own rows with the two inverted 64 x 64 diagonal blocks.
//
// Blocks are handed out bottom-up by a counter (an int in the unused lower
// part of T's first block, zero after trinv_kernel), so a workgroup waits only
// for workgroups that took their block before it, i.e. that already run: every
// wait ends whatever the order and number of resident workgroups.  X itself
// carries the hand-over: trinv_kernel has set it to kUnset (a NaN pattern that
// is never stored as a result), the owner stores its x with device-scope
// stores, and readers poll those values with device-scope loads, so no fence
// or flag is needed.  The polls are bounded all the same (a caller that lets
// two solves share one workspace gets non-finite x, not a hang).
//
// 128 rows a workgroup: the hand-over between workgroups costs more than the
// arithmetic of a block, and 128 halves their number against 64.  R's tile for
// block j - 1 is requested before x_j is awaited.  n = 4096, one right-hand
// side: 66 us against 680 us for one launch per 64-row block (64 launches of
// 10.2 us and their gaps); about 2 us per hand-over.
constexpr int kFlowRows = 128;
constexpr int kFlowThreads = 512;
constexpr int kFlowPolls = 1 << 22;

__device__ __forceinline__ double flow_load(const double* p) {
  return __longlong_as_double(
      __hip_atomic_load(reinterpret_cast<const long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

__device__ __forceinline__ void flow_store(double* p, double x) {
  long long b = __double_as_longlong(x);
  if (b == kUnset) b = 0x7ff8000000000000ll;    // a NaN all the same
  __hip_atomic_store(reinterpret_cast<long long*>(p), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Thread (lane, wave) of the flow kernel holds, of every matrix, the columns of
// its wave and row `lane` (and lane + 64 of a 128-row tile), so a vector entry
// is one LDS broadcast per wave and loads of a column of R are whole lines; the
// eight waves' sums meet in LDS.
constexpr int kFlowWaves = kFlowThreads / 64;

// acc[u] += sum over the wave's 8 columns of m[t] v[u][8 wave + t]
template <int NR>
__device__ __forceinline__ void flow_fma8(double (&acc)[NR], const double (&m)[8], const double (*v)[kFlowRows],
                                          int off) {
#pragma unroll
  for (int u = 0; u < NR; ++u)
#pragma unroll
    for (int t = 0; t < 8; t += 2) {
      const v2d x = *reinterpret_cast<const v2d*>(&v[u][off + t]);
      acc[u] += m[t] * x.x;
      acc[u] += m[t + 1] * x.y;
    }
}

// TRANS: R_1^T X = Y, the same walk from the top block down, with R's tiles and
// T transposed (a thread then holds 16 consecutive rows of columns lane and
// lane + 64; VEC: as 16-byte loads).
template <int NR, bool TRANS, bool VEC>
__global__ __launch_bounds__(kFlowThreads) void trsv_flow_kernel(const double* R, int64_t ldr, double* T,
                                                                 const double* Y, int64_t ldy, double* X, int64_t ldx,
                                                                 int nrhs, int64_t n, int nblk, int chunks) {
  __shared__ __align__(16) double xs[2][NR][kFlowRows];
  __shared__ __align__(16) double yk[NR][kFlowRows];
  __shared__ double red[kFlowWaves][NR][kFlowRows];
  __shared__ int s_ticket;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) s_ticket = atomicAdd(reinterpret_cast<int*>(T + kSolveBlock - 1), 1);
  __syncthreads();
  const int ticket = s_ticket;
  if (ticket >= nblk * chunks) return;
  const int k = TRANS ? ticket / chunks : nblk - 1 - ticket / chunks, r0 = (ticket % chunks) * NR;
  const int64_t k0 = (int64_t)k * kFlowRows;
  const int nr = nrhs - r0 < NR ? nrhs - r0 : NR;
  const bool two = k0 + kSolveBlock < n;       // the block reaches past its upper 64 rows

  // the tile of block j: rows lane and lane + 64, columns 16 wave .. 16 wave + 15
  // (TRANS: columns lane and lane + 64 of this block, rows 16 wave .. of block j;
  // blocks above another are whole)
  const double* ra = R + (k0 + lane < n ? k0 + lane : 0) + (int64_t)(16 * wave) * ldr;
  const double* rb = R + (k0 + 64 + lane < n ? k0 + 64 + lane : 0) + (int64_t)(16 * wave) * ldr;
  if (TRANS) {
    ra = R + 16 * wave + (k0 + lane < n ? k0 + lane : 0) * ldr;
    rb = R + 16 * wave + (k0 + 64 + lane < n ? k0 + 64 + lane : 0) * ldr;
  }
  auto load = [&](double (&v)[32], int j) {
    const int64_t c0 = (int64_t)j * kFlowRows;
    if constexpr (TRANS && VEC) {
#pragma unroll
      for (int t = 0; t < 16; t += 2) {
        const v2d xa = *reinterpret_cast<const v2d*>(ra + c0 + t), xb = *reinterpret_cast<const v2d*>(rb + c0 + t);
        v[t] = xa.x;
        v[t + 1] = xa.y;
        v[16 + t] = xb.x;
        v[17 + t] = xb.y;
      }
    } else if constexpr (TRANS) {
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        v[t] = ra[c0 + t];
        v[16 + t] = rb[c0 + t];
      }
    } else if (c0 + kFlowRows <= n) {
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        v[t] = ra[(c0 + t) * ldr];
        v[16 + t] = rb[(c0 + t) * ldr];
      }
    } else {
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const bool in = c0 + 16 * wave + t < n;
        v[t] = in ? ra[(c0 + t) * ldr] : 0.0;
        v[16 + t] = in ? rb[(c0 + t) * ldr] : 0.0;
      }
    }
  };
  double va[32], vb[32];
  const int first = TRANS ? 0 : nblk - 1, step = TRANS ? 1 : -1;
  const int steps = TRANS ? k : nblk - 1 - k;      // blocks solved before this one
  if (steps > 0) load(va, first);
  // the two inverted diagonal blocks and R_1[upper 64 rows, lower 64 columns]:
  // row `lane`, columns 8 wave .. 8 wave + 7 (TRANS: of their transposes); T's entries below its diagonal
  // are zero (one of them holds the counter)
  double ta[8], tb[8], rab[8];
  {
    const double* t0 = T + (k0 / kSolveBlock) * kSolveBlock * kSolveBlock;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = 8 * wave + e;
      const int i = TRANS ? c : lane, l = TRANS ? lane : c;      // the entry's row and column
      ta[e] = i <= l ? t0[i + l * kSolveBlock] : 0.0;
      tb[e] = two && i <= l ? t0[kSolveBlock * kSolveBlock + i + l * kSolveBlock] : 0.0;
      rab[e] = k0 + kSolveBlock + l < n ? R[k0 + i + (k0 + kSolveBlock + l) * ldr] : 0.0;
    }
  }
  // hand-over and the block's own rows: thread (row pr, right-hand side pu)
  const int pr = tid & (kFlowRows - 1), pu = tid / kFlowRows;
  const double y0 = (pu < nr && k0 + pr < n) ? Y[k0 + pr + (int64_t)(r0 + pu) * ldy] : 0.0;

  double aa[NR], ab[NR];
#pragma unroll
  for (int u = 0; u < NR; ++u) aa[u] = ab[u] = 0.0;
  int budget = kFlowPolls;
  auto await = [&](int j) {
    if (pu < NR) {
      const int64_t r = (int64_t)j * kFlowRows + pr;
      double x = 0.0;
      if (r < n && pu < nr) {
        const double* p = X + r + (int64_t)(r0 + pu) * ldx;
        x = flow_load(p);
        while (__double_as_longlong(x) == kUnset && budget > 0) {
          --budget;
          x = flow_load(p);
        }
      }
      xs[j & 1][pu][pr] = x;
    }
    __syncthreads();
  };
  auto subtract = [&](const double (&v)[32], int j) {
#pragma unroll
    for (int u = 0; u < NR; ++u)
#pragma unroll
      for (int t = 0; t < 16; t += 2) {
        const v2d x = *reinterpret_cast<const v2d*>(&xs[j & 1][u][16 * wave + t]);
        aa[u] += v[t] * x.x;
        ab[u] += v[16 + t] * x.x;
        aa[u] += v[t + 1] * x.y;
        ab[u] += v[17 + t] * x.y;
      }
  };
  for (int e = 0; e < steps; e += 2) {
    const int j = first + step * e;
    if (e + 1 < steps) load(vb, j + step);
    __builtin_amdgcn_sched_barrier(0);
    await(j);
    subtract(va, j);
    if (e + 1 < steps) {
      if (e + 2 < steps) load(va, j + 2 * step);
      __builtin_amdgcn_sched_barrier(0);
      await(j + step);
      subtract(vb, j + step);
    }
  }
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    red[wave][u][lane] = aa[u];
    red[wave][u][64 + lane] = ab[u];
  }
  __syncthreads();
  if (pu < NR) {                // row pr, right-hand side pu
    double y = y0;
#pragma unroll
    for (int e = 0; e < kFlowWaves; ++e) y -= red[e][pu][pr];
    yk[pu][pr] = k0 + pr < n ? y : 0.0;     // (rows past n hold sums of clamped loads)
  }
  __syncthreads();
  // x_b = T_b y_b;  y_a -= R_ab x_b;  x_a = T_a y_a (TRANS: x_a first)
  auto matvec = [&](const double (&m)[8], const double (*v)[kFlowRows], int off) {
    double s[NR];
#pragma unroll
    for (int u = 0; u < NR; ++u) s[u] = 0.0;
    flow_fma8<NR>(s, m, v, off + 8 * wave);
#pragma unroll
    for (int u = 0; u < NR; ++u) red[wave][u][lane] = s[u];
    __syncthreads();
    double x = 0.0;
    if (pu < NR && pr < kSolveBlock) {
#pragma unroll
      for (int e = 0; e < kFlowWaves; ++e) x += red[e][pu][pr];
    }
    return x;                   // of row pr < 64, right-hand side pu
  };
  // solve 64 rows (h = 0: upper, 1: lower) with their inverted block
  const bool mine = pu < NR && pr < kSolveBlock;
  auto solve = [&](const double (&m)[8], int h) {
    const double x = matvec(m, yk, kSolveBlock * h);
    if (mine) {
      xs[0][pu][pr] = x;
      const int64_t r = k0 + kSolveBlock * h + pr;
      if (r < n && pu < nr) flow_store(X + r + (int64_t)(r0 + pu) * ldx, x);
    }
    __syncthreads();
  };
  const int h0 = TRANS ? 0 : 1;
  if (TRANS || two) {
    if (TRANS) solve(ta, 0); else solve(tb, 1);
    if (!two) return;
    const double d = matvec(rab, xs[0], 0);
    if (mine) yk[pu][kSolveBlock * (1 - h0) + pr] -= d;
    __syncthreads();
  }
  if (TRANS) solve(tb, 1); else solve(ta, 0);
}

void launch_gemv_t(const double* Q, int64_t ldq, int64_t m, int n, const double* B, int64_t ldb, int nrhs,
                   double* Y, int64_t ldy, hipStream_t st) {
  // four waves per column while that keeps the grid within 1024 workgroups
  // (n = 4096: one wave per column already reads at the rate of a large copy)
  const int per = kSolveThreads / 64;
  if (n <= 1024)
    hipLaunchKernelGGL(gemv_t_kernel<4>, dim3(n), dim3(kSolveThreads), 0, st, Q, ldq, m, n, B, ldb, nrhs, Y, ldy);
  else
    hipLaunchKernelGGL(gemv_t_kernel<1>, dim3((n + per - 1) / per), dim3(kSolveThreads), 0, st, Q, ldq, m, n, B, ldb,
                       nrhs, Y, ldy);
}

void launch_trinv(const double* R, int64_t ldr, int64_t n, double* T, hipStream_t st, double* X, int64_t ldx,
                  int nrhs) {
  hipLaunchKernelGGL(trinv_kernel, dim3((unsigned)((n + kSolveBlock - 1) / kSolveBlock)), dim3(kSolveThreads), 0,
                     st, R, ldr, n, T, X, ldx, nrhs);
}

void launch_trsv_flow(const double* R, int64_t ldr, double* T, const double* Y, int64_t ldy, double* X, int64_t ldx,
                      int nrhs, int64_t n, bool trans, hipStream_t st) {
  const int nblk = (int)((n + kFlowRows - 1) / kFlowRows);
  auto go = [&](auto kern, int per) {
    const int chunks = (nrhs + per - 1) / per;
    hipLaunchKernelGGL(kern, dim3((unsigned)nblk * chunks), dim3(kFlowThreads), 0, st, R, ldr, T, Y, ldy, X, ldx, nrhs,
                       n, nblk, chunks);
  };
  const bool vec = reinterpret_cast<uintptr_t>(R) % 16 == 0 && ldr % 2 == 0;
  // one right-hand side by itself: a quarter of the LDS reads on the chain
  if (nrhs == 1) {
    if (!trans) go(trsv_flow_kernel<1, false, false>, 1);
    else if (vec) go(trsv_flow_kernel<1, true, true>, 1);
    else go(trsv_flow_kernel<1, true, false>, 1);
  } else {
    if (!trans) go(trsv_flow_kernel<kRhsChunk, false, false>, kRhsChunk);
    else if (vec) go(trsv_flow_kernel<kRhsChunk, true, true>, kRhsChunk);
    else go(trsv_flow_kernel<kRhsChunk, true, false>, kRhsChunk);
  }
}

// Scratch memory of the allocation-free solve (coded_qr_solve_noalloc): the
// inverted diagonal blocks of R_1 and Y = Qpost^T Bpost live in this
// file-scope array, one copy per device, held until the process ends.  Host
// code never passes the array's name to a kernel (on the host it is only a
// stand-in for the symbol): its device address is looked up once per device,
// with that device current, and that address is what the kernels receive.
// Every kernel writes the parts of it that later kernels read (trinv_kernel
// all 64 x 64 entries of each block, the counter among them, gemv_t_kernel
// all n x nrhs entries of Y), so no call depends on what a previous call left there.
static __device__ __align__(256) char scratch[kSolveScratchBytes];

hipError_t solve_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* a = nullptr;
    e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = a;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

}  // namespace cqr
