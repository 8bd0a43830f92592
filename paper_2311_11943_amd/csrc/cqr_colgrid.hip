// The column-wise panel leaf (CGS2, ICGS, MGS) of the reduced-precision modes,
// two launches per column (one for MGS).  FP64 factorizations take
// colstep_kernel / colmgs_kernel (cqr_gemm.hip), which are twice as fast; the
// reduced-precision modes keep this one for its order of sums: their
// coefficients are rounded from the column state, so a rounding-level change of
// a panel moves them by an FP32 rounding here and there, and the R blocks decoded
// from unfinished columns by up to 1e-7 of an entry (n = 1632, FP32
// coefficients, one failure event), more than any FP64 result moves.
#include "cqr_colwise.hpp"
#include "cqr_kernels.hpp"

#include <algorithm>
#include <cmath>

namespace cqr {

// A panel leaf orthogonalised column by column (the CGS2, ICGS and MGS panel
// modes) by a grid of workgroups, each owning one slab of rows.  A column
// needs a sum over all rows before every update, so each step of the method
// is one launch: it first reduces the partial sums every workgroup of the
// previous launch left (all workgroups sum them redundantly, in the same
// fixed order, so they take identical decisions), then works on its own
// slab and leaves its partial sums for the next launch.  Kernel boundaries
// order the steps; nothing waits inside a launch.
//
// CGS2 / ICGS, column j:
//   PROJECT(j)  s1 = the reduced P[:, <j]^T p_j; column j-1 normalised by its
//               r (known now); p_j -= P[:, <j] s1; partials of ||p_j||^2 and,
//               speculatively, of P[:, <j]^T p_j for a second projection.
//   REORTH(j)   second projection when CGS2, or when ICGS finds
//               ||p_j||^2 < eta^2 ||p_j before||^2 (the DGKS test); partials
//               of ||p_j||^2, of ||p_{j+1}||^2 and of P[:, <=j]^T p_{j+1}
//               (column j not yet normalised: that product is divided by
//               r_jj in PROJECT(j+1)).
// MGS, column i (the paper's sequential MGS):
//   MGS(i)      r_{i-1,i-1} and r_{i-1,c} = u_{i-1}^T u_c / r_{i-1,i-1} from
//               the reduced sums; q_{i-1} = u_{i-1} / r_{i-1,i-1};
//               u_c -= r_{i-1,c} q_{i-1} for c >= i; partials of ||u_i||^2 and
//               of u_i^T u_c for c > i.
// FINISH normalises the last column.  Workgroup 0 writes R.
//
// A thread loads the columns a step touches in its row into registers at
// once (the first row block before the reduction of the previous partial
// sums, so that the two memory latencies overlap), computes the update and
// the step's inner products from them, and stores what changed; one row per
// thread up to 65536 rows.  The wavefront sums of every 16-slot chunk are
// formed first and exchanged through LDS once per row block.  Partial sums:
// slots [0, 64) inner products (whole 16-slot chunks are written), 64-66 the
// squared norms (all three written by every launch).
constexpr int kGridMax = 256;
constexpr int kGridSlots = 68;       // 64 inner products, three squared norms, one spare
static_assert(2 * (int64_t)kGridMax * kGridSlots + 4 <= kColWorkDoubles, "scratch");
enum : int { CG_START = 0, CG_PROJECT = 1, CG_REORTH = 2, CG_FINISH = 3, CG_MGS = 4 };
constexpr int kGridThreads = 256;
constexpr int kSlotNA = 64, kSlotNB = 65, kSlotNC = 66;

// Row r's columns [lo, hi) into v (zeros elsewhere) and its columns e0 and
// e1 (e1 < 0: none) into x0, x1, addressed as a uniform column base plus the
// row's 32-bit byte offset in the slab that starts at row r0.
__device__ __forceinline__ void colgrid_load_row(double (&v)[kLeaf], double& x0, double& x1, const double* P,
                                                 int64_t r0, int64_t ld, int64_t r, bool act, int lo, int hi, int e0,
                                                 int e1) {
  const char* const slab = reinterpret_cast<const char*>(P + r0);
  const uint32_t off = act ? (uint32_t)(r - r0) * 8u : 0u;
#pragma unroll
  for (int c = 0; c < kLeaf; ++c)
    v[c] = (act && c >= lo && c < hi) ? *reinterpret_cast<const double*>(slab + c * ld * 8 + off) : 0.0;
  x0 = act ? P[r + e0 * ld] : 0.0;
  x1 = act && e1 >= 0 ? P[r + e1 * ld] : 0.0;
}

template <int kind>
__global__ __launch_bounds__(kGridThreads) void colgrid_kernel(ColArgs a, int G, int64_t rb, int j, int par) {
  __builtin_amdgcn_s_setprio(2);   // panel chain
  __shared__ double red[kGridSlots];
  __shared__ double tmp[kGridThreads];
  __shared__ double wsum[kGridThreads / 64][kLeaf + kColChunk];   // per-wavefront sums of every slot
  __shared__ double coef[kLeaf + kColChunk];                     // zero beyond the step's coefficients
  const int tid = threadIdx.x, g = blockIdx.x, w = a.w;
  const int64_t ld = a.ldp;
  double* const P = a.P;
  const int64_t r0 = (int64_t)g * rb, r1 = min(a.mrows, r0 + rb);
  const int64_t bufsz = (int64_t)kGridMax * kGridSlots;
  const double* in = a.work + (par ^ 1) * bufsz;
  double* out = a.work + par * bufsz + (int64_t)g * kGridSlots;
  double* state = a.work + 2 * bufsz;   // [0] ||p_j||^2 before its first projection, [1] after it, [2] second taken
  const bool lead = g == 0 && tid == 0;

  // inner-product slots this launch reads [rlo, rhi) and writes [wlo, whi);
  // columns a row holds in registers [lo, hi); single columns e0 and e1
  int rlo = 0, rhi = 0, wlo = 0, whi = 0, lo = 0, hi = 0, e0 = 0, e1 = -1;
  if constexpr (kind == CG_PROJECT) {   // e0 = p_j, e1 = column j-1
    rhi = j; whi = j; hi = j; e0 = j; e1 = j - 1;
  }
  if constexpr (kind == CG_REORTH) {    // e0 = p_j, e1 = p_{j+1}
    rhi = j; whi = j + 1 < w ? j + 1 : 0; hi = j; e0 = j; e1 = j + 1 < w ? j + 1 : -1;
  }
  if constexpr (kind == CG_MGS) {       // e0 = u_j, e1 = u_{j-1}
    if (j > 0) { rlo = j; rhi = w; }
    wlo = j + 1; whi = w; lo = j; hi = w; e0 = j; e1 = j - 1;
  }
  if constexpr (kind == CG_FINISH) e0 = w - 1;

  double v[kLeaf], x0 = 0.0, x1 = 0.0;
  // the first row block is loaded before the reduction below, which it does
  // not depend on, so the two memory latencies overlap
  const int nit = (int)((rb + kGridThreads - 1) / kGridThreads);
  colgrid_load_row(v, x0, x1, P, r0, ld, r0 + tid, r0 + tid < r1, lo, hi, e0, e1);
  // the state words a step uses, read before the reduction below (workgroup 0
  // of the same launch writes only words the step does not read: PROJECT
  // writes [0] and reads [1], [2]; REORTH writes [1], [2] and reads [0])
  double st0 = 0.0, st1 = 0.0, st2 = 0.0;
  if constexpr (kind == CG_REORTH) st0 = state[0];
  if constexpr (kind == CG_PROJECT || kind == CG_FINISH) {
    st1 = state[1];
    st2 = state[2];
  }

  for (int c = tid; c < kLeaf + kColChunk; c += kGridThreads) coef[c] = 0.0;
  // reduce the previous launch's partials: its inner products in [rlo, rhi)
  // and the three norms; thread (si, q) sums workgroups q, q + Q, ... in order
  if (!(kind == CG_START || (kind == CG_MGS && j == 0))) {
    const int nd = rhi - rlo, ns = nd + 3, Q = kGridThreads / ns;
    const int si = tid % ns, q = tid / ns;
    const int slot = si < nd ? rlo + si : kSlotNA + (si - nd);
    if (q < Q) {
      double acc = 0.0;
      int h = q;
      for (; h + 3 * Q < G; h += 4 * Q) {
        const double y0 = in[(int64_t)h * kGridSlots + slot], y1 = in[(int64_t)(h + Q) * kGridSlots + slot];
        const double y2 = in[(int64_t)(h + 2 * Q) * kGridSlots + slot], y3 = in[(int64_t)(h + 3 * Q) * kGridSlots + slot];
        acc += y0;
        acc += y1;
        acc += y2;
        acc += y3;
      }
      for (; h < G; h += Q) acc += in[(int64_t)h * kGridSlots + slot];
      tmp[q * ns + si] = acc;
    }
    __syncthreads();
    if (tid < ns) {
      double s = 0.0;
      for (int k = 0; k < Q; ++k) s += tmp[k * ns + tid];
      red[tid < nd ? rlo + tid : kSlotNA + (tid - nd)] = s;
    }
  }
  __syncthreads();
  // r from a squared norm; a zero or non-finite norm flags the panel as
  // exactly rank-deficient and leaves the column unnormalised
  auto diag = [&](double r2) {
    if (!(r2 > 0.0) || !isfinite(r2)) {
      if (lead && a.info[0] == 0) a.info[0] = 1 + a.panel;
      r2 = 1.0;
    }
    return sqrt(r2);
  };

  if constexpr (kind == CG_FINISH) {
    // r of the last column, which is normalised; zeros below R's diagonal
    const double r = diag(a.mode == COLWISE_MGS ? red[kSlotNA] : (st2 != 0.0 ? red[kSlotNC] : st1));
    const double inv = 1.0 / r;
    if (lead) a.Rout[(w - 1) + (int64_t)(w - 1) * a.ldr] = r;
    if (g == 0)
      for (int e = tid; e < w * w; e += kGridThreads) {
        const int i = e % w, c = e / w;
        if (i > c) a.Rout[i + (int64_t)c * a.ldr] = 0.0;
      }
    for (int it = 0; it < nit; ++it) {
      const int64_t r = r0 + (int64_t)it * kGridThreads + tid;
      if (it > 0) colgrid_load_row(v, x0, x1, P, r0, ld, r, r < r1, lo, hi, e0, e1);
      if (r < r1) P[r + (w - 1) * ld] = x0 * inv;
    }
  } else {
    // this step's coefficients, decision and R entries
    double inv = 1.0;
    bool second = false;
    if constexpr (kind == CG_PROJECT) {
      if (j > 0) {
        const double r = diag(st2 != 0.0 ? red[kSlotNC] : st1);
        inv = 1.0 / r;
        if (lead) a.Rout[(j - 1) + (int64_t)(j - 1) * a.ldr] = r;
      }
      if (tid < j) coef[tid] = tid == j - 1 ? red[tid] * inv : red[tid];
      __syncthreads();
      if (g == 0) {
        if (tid < j) a.Rout[tid + (int64_t)j * a.ldr] = coef[tid];
        if (tid == 0) state[0] = red[kSlotNA];
      }
    } else if constexpr (kind == CG_REORTH) {
      const double n1 = red[kSlotNB];
      second = j > 0 && (a.mode == COLWISE_CGS2 || n1 < a.eta * a.eta * st0);
      if (second && tid < j) coef[tid] = red[tid];
      __syncthreads();
      if (g == 0) {
        if (second && tid < j) a.Rout[tid + (int64_t)j * a.ldr] += coef[tid];
        if (tid == 0) {
          state[1] = n1;
          state[2] = second ? 1.0 : 0.0;
        }
      }
    } else if constexpr (kind == CG_MGS) {
      if (j > 0) {
        const double r = diag(red[kSlotNA]);
        inv = 1.0 / r;
        if (tid >= j && tid < w) coef[tid] = red[tid] * inv;
        if (lead) a.Rout[(j - 1) + (int64_t)(j - 1) * a.ldr] = r;
      }
      __syncthreads();
      if (g == 0 && j > 0 && tid >= j && tid < w) a.Rout[(j - 1) + (int64_t)tid * a.ldr] = coef[tid];
    }

    double total = 0.0;   // threads < kGridSlots: this workgroup's sum for slot tid
    for (int it = 0; it < nit; ++it) {
      const int64_t r = r0 + (int64_t)it * kGridThreads + tid;
      const bool act = r < r1;
      if (it > 0) colgrid_load_row(v, x0, x1, P, r0, ld, r, act, lo, hi, e0, e1);
      double na = 0.0, nb = 0.0, nc = 0.0;
      if constexpr (kind == CG_START) {
        na = x0 * x0;
      } else if constexpr (kind == CG_PROJECT) {
        // column j-1 normalised; p_j -= P[:, <j] s1; ||p_j||^2; P[:, <j]^T p_j
        double x = x0;
        if (j > 0) {
          const double qp = x1 * inv;
          if (act) P[r + (j - 1) * ld] = qp;
#pragma unroll
          for (int c = 0; c < kLeaf; ++c)
            if (c + 1 == j) v[c] = qp;
        }
#pragma unroll
        for (int c = 0; c < kLeaf; ++c) x -= v[c] * coef[c];
        if (act) P[r + j * ld] = x;
        nb = x * x;
#pragma unroll
        for (int c = 0; c < kLeaf; ++c) v[c] *= x;
      } else if constexpr (kind == CG_REORTH) {
        double x = x0;
        const double y = x1;
        if (second) {
#pragma unroll
          for (int c = 0; c < kLeaf; ++c) x -= v[c] * coef[c];
          if (act) P[r + j * ld] = x;
          nc = x * x;
        }
        // the next column's first projection: P[:, <=j]^T p_{j+1}, ||p_{j+1}||^2
        na = y * y;
#pragma unroll
        for (int c = 0; c < kLeaf; ++c) v[c] = c == j ? x * y : v[c] * y;
      } else {   // CG_MGS
        // q_{j-1} = u_{j-1} / r; u_c -= r_{j-1,c} q_{j-1} for c >= j;
        // ||u_j||^2 and u_j^T u_c for c > j
        double u = x0;
        if (j > 0) {
          const double q = x1 * inv;
          if (act) P[r + (j - 1) * ld] = q;
          u -= coef[j] * q;
          const uint32_t off = act ? (uint32_t)(r - r0) * 8u : 0u;
          char* const wslab = reinterpret_cast<char*>(P + r0);
#pragma unroll
          for (int c = 0; c < kLeaf; ++c) {
            v[c] -= coef[c] * q;
            if (act && c >= j && c < w) *reinterpret_cast<double*>(wslab + c * ld * 8 + off) = v[c];
          }
        }
        na = u * u;
#pragma unroll
        for (int c = 0; c < kLeaf; ++c) v[c] *= u;
      }
      // workgroup sums of this row block (the chunks covering [wlo, whi),
      // then the norms): every wavefront butterfly first, independent of one
      // another, then one exchange through LDS; each slot's total adds the
      // wavefronts in order, then the row blocks in order
      double xs[kLeaf / kColChunk + 1];
#pragma unroll
      for (int k = 0; k < kLeaf / kColChunk; ++k) {
        xs[k] = 0.0;
        if (whi > wlo && (k + 1) * kColChunk > wlo && k * kColChunk < whi) {
          double v16[kColChunk];
#pragma unroll
          for (int c = 0; c < kColChunk; ++c) v16[c] = v[k * kColChunk + c];
          xs[k] = colwise_wave_sum16(v16);
        }
      }
      {
        double n16[kColChunk];
#pragma unroll
        for (int c = 0; c < kColChunk; ++c) n16[c] = 0.0;
        n16[0] = na;
        n16[1] = nb;
        n16[2] = nc;
        xs[kLeaf / kColChunk] = colwise_wave_sum16(n16);
      }
      const int wave = tid >> 6, lane = tid & 63;
      if (lane < kColChunk) {
#pragma unroll
        for (int k = 0; k <= kLeaf / kColChunk; ++k) wsum[wave][k * kColChunk + lane] = xs[k];
      }
      __syncthreads();
      if (tid < kGridSlots) {
        double sacc = 0.0;
#pragma unroll
        for (int q = 0; q < kGridThreads / 64; ++q) sacc += wsum[q][tid];
        total += sacc;
      }
      __syncthreads();
    }
    const int k = tid / kColChunk;
    const bool chunk = whi > wlo && (k + 1) * kColChunk > wlo && k * kColChunk < whi && tid < kLeaf;
    if (chunk || (tid >= kSlotNA && tid <= kSlotNC)) out[tid] = total;
  }
}

// The launches of one leaf: 2w + 2 for CGS2 / ICGS, w + 1 for MGS.  One row
// per thread while the rows fit kGridMax workgroups, more beyond.
void launch_colgrid(const ColArgs& a, hipStream_t st) {
  const int G = (int)std::min<int64_t>(kGridMax, std::max<int64_t>(1, (a.mrows + kGridThreads - 1) / kGridThreads));
  const int64_t rb = (a.mrows + G - 1) / G;
  int par = 0;
  auto go = [&](auto kern, int j) {
    hipLaunchKernelGGL(kern, dim3(G), dim3(kGridThreads), 0, st, a, G, rb, j, par);
    par ^= 1;
  };
  if (a.mode == COLWISE_MGS) {
    for (int i = 0; i < a.w; ++i) go(colgrid_kernel<CG_MGS>, i);
  } else {
    go(colgrid_kernel<CG_START>, 0);
    for (int j = 0; j < a.w; ++j) {
      go(colgrid_kernel<CG_PROJECT>, j);
      go(colgrid_kernel<CG_REORTH>, j);
    }
  }
  go(colgrid_kernel<CG_FINISH>, a.w - 1);
}

}  // namespace cqr
