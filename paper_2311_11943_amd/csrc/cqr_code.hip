// Memory-bound kernels of the code: encoding, erasure (failure simulation),
// decoding / re-encoding along code lines, post-orthogonalization.
// Consecutive threads take consecutive rows of a column-major matrix, so every
// wavefront load and store covers whole 128-byte lines.
#include "cqr_kernels.hpp"

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

namespace cqr {

constexpr int kThreads = 256;

static unsigned grid_for(int64_t n) {
  int64_t b = (n + kThreads - 1) / kThreads;
  return (unsigned)(b < 1 ? 1 : b);
}

// --------------------------------------------------------------------------
// Checksum rows alone, C_(k,J) = sum_t g~_v[k][t] A_(t,J) for all n columns
// (R's vertical code when the plan has no horizontal code).  Thread = (row r
// in a block, column c).
// --------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void encode_rows_kernel(EncodeArgs a) {
  int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= a.bs * a.n) return;
  int64_t r = e % a.bs, c = e / a.bs;
  double* col = a.At + c * a.ld;
  double acc[kMaxGen];
#pragma unroll
  for (int k = 0; k < kMaxGen; ++k) acc[k] = 0.0;
  for (int t = 0; t < a.pr; ++t) {
    double v = col[t * a.bs + r];
#pragma unroll
    for (int k = 0; k < kMaxGen; ++k)
      if (k < a.kv) acc[k] += a.g[k * a.pr + t] * v;
  }
#pragma unroll
  for (int k = 0; k < kMaxGen; ++k)
    if (k < a.kv) col[a.m + k * a.bs + r] = acc[k];
}

// --------------------------------------------------------------------------
// Encode in one pass (the whole encoding equation): checksum rows, checksum
// columns and corner from a single read of A.  A workgroup takes R = 512 / T
// consecutive rows r of a block row at one column position s of a block
// column, and walks the p_r block rows u; thread (rho, t) loads the element
// at row u bs + r, column t bw + s for every u up front (all its loads in
// flight at once), and
//   - as a row-code thread (t < p_c) sums C_k += g~_v[k][u] A_(u,t)[r, s]
//     over u (checksum block row k, block column t);
//   - as a column-code thread (t = l < K_h) forms, for each u, the checksum
//     column entry sum_t' g~_h[t'][l] A_(u,t')[r, s] from the workgroup's
//     LDS copy of that row of blocks, and after the walk the corner entries
//     sum_t' g~_h[t'][l] C_k(t') from the row-code threads' sums.
// Threads (rho, t) with the same t read R consecutive rows of one column:
// whole cache-line segments per wave and column.  Every element of A is read
// once and every checksum element written once: 8 (mn + cn + md + cd) bytes.
// 512 threads: at p_c = 16, 32-row (256-byte) segments per column; alone, on
// the n = 32768 workload's encode (18 GB), 3.97 TB/s against 3.66 with 256
// threads (16-row segments) and 3.25 with 1024.
// --------------------------------------------------------------------------
constexpr int kEncThreads = 512;

template <int T>
__global__ __launch_bounds__(kEncThreads) void encode_fused_kernel(EncodeArgs a) {
  constexpr int R = kEncThreads / T;
  __shared__ double X[2][T][R + 1];
  __shared__ double Cl[kMaxGen][T][R + 1];
  __shared__ double Gc[kMaxGen][kMaxGrid];
  const int tid = threadIdx.x, rho = tid % R, t = tid / R;
  const int64_t nseg = (a.bs + R - 1) / R;
  const int64_t s = blockIdx.x / nseg;
  const int64_t r = (blockIdx.x % nseg) * R + rho;
  const bool rok = r < a.bs;
  const bool rowt = t < a.pc, colt = t < a.kh;
  for (int e = tid; e < kMaxGen * kMaxGrid; e += kEncThreads) Gc[e / kMaxGrid][e % kMaxGrid] = a.gc[e];
  double x[kMaxGrid];
  const double* src = a.At + r + (t * a.bw + s) * a.ld;
#pragma unroll
  for (int u = 0; u < kMaxGrid; ++u) x[u] = (u < a.pr && rok && rowt) ? src[u * a.bs] : 0.0;
  double c[kMaxGen];
#pragma unroll
  for (int k = 0; k < kMaxGen; ++k) c[k] = 0.0;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kMaxGrid; ++u) {
    if (u >= a.pr) break;
    X[u & 1][t][rho] = x[u];
#pragma unroll
    for (int k = 0; k < kMaxGen; ++k)
      if (k < a.kv) c[k] += a.g[k * a.pr + u] * x[u];
    __syncthreads();
    if (colt && rok) {
      double d = 0.0;
      for (int tt = 0; tt < a.pc; ++tt) d += Gc[t][tt] * X[u & 1][tt][rho];
      a.At[u * a.bs + r + (a.n + t * a.bw + s) * a.ld] = d;
    }
  }
  if (a.kv == 0) return;
  if (rowt) {
#pragma unroll
    for (int k = 0; k < kMaxGen; ++k)
      if (k < a.kv) {
        Cl[k][t][rho] = c[k];
        if (rok) a.At[a.m + k * a.bs + r + (t * a.bw + s) * a.ld] = c[k];
      }
  }
  __syncthreads();
  if (colt && rok) {
    for (int k = 0; k < a.kv; ++k) {
      double e = 0.0;
      for (int tt = 0; tt < a.pc; ++tt) e += Gc[t][tt] * Cl[k][tt][rho];
      a.At[a.m + k * a.bs + r + (a.n + t * a.bw + s) * a.ld] = e;
    }
  }
}

void launch_encode_fused(const EncodeArgs& a, hipStream_t st) {
  const int T = std::max(a.pc, a.kh) <= 8 ? 8 : (std::max(a.pc, a.kh) <= 16 ? 16 : 32);
  const int R = kEncThreads / T;
  const unsigned grid = (unsigned)(((a.bs + R - 1) / R) * a.bw);
  if (T == 8)
    hipLaunchKernelGGL(encode_fused_kernel<8>, dim3(grid), dim3(kEncThreads), 0, st, a);
  else if (T == 16)
    hipLaunchKernelGGL(encode_fused_kernel<16>, dim3(grid), dim3(kEncThreads), 0, st, a);
  else
    hipLaunchKernelGGL(encode_fused_kernel<32>, dim3(grid), dim3(kEncThreads), 0, st, a);
}

void launch_encode_rows(const EncodeArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(encode_rows_kernel, dim3(grid_for(a.bs * a.n)), dim3(kThreads), 0, st, a);
}

// A block of rows x cols elements, V consecutive rows a thread: consecutive
// threads go down a column and on into the next, so that every thread of every
// workgroup but the last has rows, whatever the block's height (runs of 512 rows
// left a third of the threads without any at 672 rows).
static unsigned block_grid(int rows, int cols, int V) {
  return (unsigned)(((int64_t)rows / V * cols + kThreads - 1) / kThreads);
}

// first row and column of this thread in workgroup b
__device__ __forceinline__ void block_pos(int rows, unsigned b, int V, int& r, int& c) {
  const unsigned per = (unsigned)rows / V;
  const uint64_t e = (uint64_t)b * kThreads;
  const unsigned c0 = (unsigned)(e >> 32 ? e / per : (unsigned)e / per);     // (uniform)
  const unsigned t = (unsigned)(e - (uint64_t)c0 * per) + threadIdx.x, q = t / per;
  r = (int)((t - q * per) * V);
  c = (int)(c0 + q);
}

// --------------------------------------------------------------------------
// Code lines: every output block of a line is a fixed linear combination of
// the line's surviving blocks (coefficients solved on the host).  Several lines
// share a launch (grid y).  Bound by HBM; a thread takes V consecutive rows of
// all blocks of its line and requests eight sources (four for a remainder of up
// to four) before it uses the first (one launch per line with one load in flight
// per thread: 58 MB in 18 us; the n = 8192 storm, 16 x 16 grid, 40 lines: erasure
// and recovery 866 us, now 500, 4.6 TB/s; one lost node, n = 8190 on 7 x 5: 53
// us, now 45).
// --------------------------------------------------------------------------
template <int V, class Args>
__global__ __launch_bounds__(kThreads) void lines_kernel(Args a) {
  typedef double vec __attribute__((ext_vector_type(V)));
  constexpr bool kOne = sizeof(a.line) == sizeof(LineSpec);       // (its line read without an index)
  const LineSpec& L = a.line[kOne ? 0 : blockIdx.y];
  int r, c;
  block_pos(a.rows, blockIdx.x, V, r, c);
  if (c >= a.cols) return;
  double* base = a.base + L.off + r + (int64_t)c * a.ld;
  const double* coef = a.coef + L.coef;
  const int ns = L.nsrc;
  double acc[kMaxOut][V];
#pragma unroll
  for (int o = 0; o < kMaxOut; ++o)
#pragma unroll
    for (int e = 0; e < V; ++e) acc[o][e] = 0.0;
  auto batch = [&](auto n, int s0) {
    constexpr int kBatch = decltype(n)::value;
    vec v[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k)      // (past the last source: its block again, not used)
      v[k] = *reinterpret_cast<const vec*>(base + L.src[min(s0 + k, ns - 1)] * a.slot);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int o = 0; o < kMaxOut; ++o) {
      if (o >= L.nout) break;
      const double* co = coef + o * ns + s0;
#pragma unroll
      for (int k = 0; k < kBatch; ++k)
        if (s0 + k < ns) {
          const double w = co[k];
#pragma unroll
          for (int e = 0; e < V; ++e) acc[o][e] += w * v[k][e];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  int s0 = 0;
  for (; ns - s0 > 4; s0 += 8) batch(std::integral_constant<int, 8>{}, s0);
  if (s0 < ns) batch(std::integral_constant<int, 4>{}, s0);
#pragma unroll
  for (int o = 0; o < kMaxOut; ++o)
    if (o < L.nout) {
      vec x;
#pragma unroll
      for (int e = 0; e < V; ++e) x[e] = acc[o][e];
      *reinterpret_cast<vec*>(base + L.dst[o] * a.slot) = x;
    }
}

// two rows a thread where every block starts 16-byte aligned and has an even
// number of rows
static bool even_blocks(const double* base, int64_t ld, int rows, int64_t slot, int64_t off) {
  return reinterpret_cast<uintptr_t>(base) % 16 == 0 && ld % 2 == 0 && rows % 2 == 0 && slot % 2 == 0 && off % 2 == 0;
}

template <class Args>
static void launch_lines_as(const Args& a, bool two, hipStream_t st) {
  const unsigned grid = block_grid(a.rows, a.cols, two ? 2 : 1);
  if (two)
    hipLaunchKernelGGL((lines_kernel<2, Args>), dim3(grid, a.nlines), dim3(kThreads), 0, st, a);
  else
    hipLaunchKernelGGL((lines_kernel<1, Args>), dim3(grid, a.nlines), dim3(kThreads), 0, st, a);
}

// a's lines and coefficients in arguments with less room
template <class Args>
static Args lines_in(const LinesArgs& a, int used) {
  Args s;
  s.base = a.base; s.ld = a.ld; s.slot = a.slot;
  s.rows = a.rows; s.cols = a.cols; s.nlines = a.nlines;
  std::copy(a.line, a.line + a.nlines, s.line);
  std::copy(a.coef, a.coef + used, s.coef);
  return s;
}

// A small event (one lost node: a line of a few blocks per matrix) is bound by
// its launches, and those by what the host writes for them, so the arguments
// have the room that the lines need, not the 6 KB of sixteen (n = 256 to 4096,
// one node erased and recovered: 30.2 us with 6 KB, 28.4 so).
static_assert(sizeof(LinesArgsOf<1, 32>) <= 384 && sizeof(LinesArgsOf<4, 256>) <= 2400 && sizeof(EraseArgsOf<16>) <= 160,
              "small arguments");
void launch_lines(const LinesArgs& a, hipStream_t st) {
  if (a.nlines <= 0) return;
  bool two = true;
  for (int l = 0; l < a.nlines; ++l) two = two && even_blocks(a.base, a.ld, a.rows, a.slot, a.line[l].off);
  const LineSpec& last = a.line[a.nlines - 1];
  const int used = last.coef + last.nsrc * last.nout;
  if (a.nlines == 1 && used <= 32)
    launch_lines_as(lines_in<LinesArgsOf<1, 32>>(a, used), two, st);
  else if (a.nlines <= 4 && used <= 256)
    launch_lines_as(lines_in<LinesArgsOf<4, 256>>(a, used), two, st);
  else
    launch_lines_as(a, two, st);
}

// Blocks set to NaN (grid y: the block); bound by its stores.
template <int V, class Args>
__global__ __launch_bounds__(kThreads) void erase_kernel(Args a) {
  typedef double vec __attribute__((ext_vector_type(V)));
  int r, c;
  block_pos(a.rows, blockIdx.x, V, r, c);
  if (c >= a.cols) return;
  *reinterpret_cast<vec*>(a.base + a.off[blockIdx.y] + r + (int64_t)c * a.ld) = __builtin_nan("");
}

template <class Args>
static void launch_erase_as(const Args& a, hipStream_t st) {
  bool two = true;
  for (int k = 0; k < a.nblk; ++k) two = two && even_blocks(a.base, a.ld, a.rows, 0, a.off[k]);
  const unsigned grid = block_grid(a.rows, a.cols, two ? 2 : 1);
  if (two)
    hipLaunchKernelGGL((erase_kernel<2, Args>), dim3(grid, a.nblk), dim3(kThreads), 0, st, a);
  else
    hipLaunchKernelGGL((erase_kernel<1, Args>), dim3(grid, a.nblk), dim3(kThreads), 0, st, a);
}

template <int BLOCKS>
static void launch_erase_in(const EraseArgs& a, hipStream_t st) {
  EraseArgsOf<BLOCKS> s;
  s.base = a.base; s.ld = a.ld; s.rows = a.rows; s.cols = a.cols; s.nblk = a.nblk;
  std::copy(a.off, a.off + a.nblk, s.off);
  launch_erase_as(s, st);
}

// (arguments with the room that the blocks need, as launch_lines)
void launch_erase(const EraseArgs& a, hipStream_t st) {
  if (a.nblk <= 0) return;
  if (a.nblk <= 16)
    launch_erase_in<16>(a, st);
  else if (a.nblk <= 64)
    launch_erase_in<64>(a, st);
  else
    launch_erase_as(a, st);
}

// --------------------------------------------------------------------------
// Post-orthogonalization  W = (G^_0 (x) I_bs) Z  (G^_0 built from G~_v) with
//   G^_0 = [[I_K + G~_1, V~], [V~^T, -I]]:
//   block row i <  K: sum_l G^_0[i][l] Z_l   (all p_r blocks)
//   block row i >= K: sum_{l<K} V~[l][i-K] Z_l - Z_i
// Thread = (row r in a block, column c); reads the p_r blocks once.
// --------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void postorth_kernel(PostArgs a) {
  int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= a.bs * a.cols) return;
  int64_t r = e % a.bs, c = e / a.bs;
  const double* src = a.src + c * a.lds + r;
  double* dst = a.dst + c * a.ldd + r;
  double z[kMaxGrid];
#pragma unroll
  for (int l = 0; l < kMaxGrid; ++l) z[l] = (l < a.pr) ? src[l * a.bs] : 0.0;
  // G^_0[i][l]: i, l < K: delta_il + G~_1[i][l];  i < K <= l: V~[i][l-K] = g~_v[i][l];
  //            i >= K > l: V~[l][i-K] = g~_v[l][i];  i, l >= K: -delta_il.
  double head[kMaxGen];
#pragma unroll
  for (int i = 0; i < kMaxGen; ++i) {
    double v = 0.0;
    if (i < a.kv) {
      v = z[i];
#pragma unroll
      for (int l = 0; l < kMaxGrid; ++l)
        if (l < a.pr) v += a.gv[i * a.pr + l] * z[l];
    }
    head[i] = v;
  }
#pragma unroll
  for (int i = 0; i < kMaxGrid; ++i) {
    if (i >= a.kv && i < a.pr) {
      double v = -z[i];
#pragma unroll
      for (int l = 0; l < kMaxGen; ++l)
        if (l < a.kv) v += a.gv[l * a.pr + i] * z[l];
      dst[i * a.bs] = v;
    }
  }
#pragma unroll
  for (int i = 0; i < kMaxGen; ++i)
    if (i < a.kv) dst[i * a.bs] = head[i];
}

void launch_postorth(const PostArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(postorth_kernel, dim3(grid_for(a.bs * a.cols)), dim3(kThreads), 0, st, a);
}

__global__ void zero_ints_kernel(int* p, int n) {
  int e = blockIdx.x * kThreads + threadIdx.x;
  if (e < n) p[e] = 0;
}

void launch_zero_ints(int* p, int n, hipStream_t st) {
  hipLaunchKernelGGL(zero_ints_kernel, dim3(grid_for(n)), dim3(kThreads), 0, st, p, n);
}

__global__ __launch_bounds__(kThreads) void fill_zero_kernel(double* p, int64_t ld, int64_t rows, int64_t cols) {
  int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= rows * cols) return;
  p[(e % rows) + (e / rows) * ld] = 0.0;
}

void launch_fill_zero(double* p, int64_t ld, int64_t rows, int64_t cols, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(rows * cols)), dim3(kThreads), 0, st, p, ld, rows, cols);
}

}  // namespace cqr
