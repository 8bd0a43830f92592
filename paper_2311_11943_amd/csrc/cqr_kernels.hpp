// Internal interface between the C-ABI layer and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace cqr {

constexpr int kMaxLine = 32;     // blocks in one code line (data + checksums)
constexpr int kMaxOut = 8;       // blocks written by one decode launch
constexpr int kMaxGen = 8;       // checksum blocks per code (K_v, K_h)
constexpr int kMaxGrid = 32;     // p_r, p_c upper bound
constexpr int kLeaf = 64;        // widest panel leaf factored by Cholesky QR
constexpr int kTile = 64;        // output tile of the split-K product kernel

// Code lines decoded by one launch.  Line l's blocks lie `slot` elements apart
// from base + off; out_o = sum_s coef[o * nsrc + s] src_s.
constexpr int kLinesMax = 16;    // lines a launch
constexpr int kLinesCoef = 640;  // coefficients a launch; one line has at most 256
struct LineSpec {
  int64_t off;
  int coef;                      // first coefficient
  uint8_t nsrc, nout;
  uint8_t src[kMaxLine];
  uint8_t dst[kMaxOut];
};
// LINES and COEF: the room for lines and coefficients (launch_lines picks what
// the kernel is given)
template <int LINES, int COEF>
struct LinesArgsOf {
  double* base;
  int64_t ld, slot;
  int rows, cols, nlines;
  LineSpec line[LINES];
  double coef[COEF];
};
typedef LinesArgsOf<kLinesMax, kLinesCoef> LinesArgs;
static_assert(kMaxOut * kMaxLine <= kLinesCoef, "a line's coefficients fit one launch");

constexpr int kEraseMax = 256;   // blocks an erasure launch
template <int BLOCKS>
struct EraseArgsOf {
  double* base;
  int64_t ld;
  int rows, cols;
  int nblk;
  int64_t off[BLOCKS];
};
typedef EraseArgsOf<kEraseMax> EraseArgs;

struct EncodeArgs {
  double* At;
  int64_t ld;
  int64_t m, n, bs, bw;
  int pr, pc, kv, kh;
  double g[kMaxGen * kMaxGrid];    // row code: g[k * pr + t] = g~_v[k][t]
  double gc[kMaxGen * kMaxGrid];   // column code: gc[l * kMaxGrid + t] = g~_h[t][l]
};

struct PostArgs {
  const double* src;
  int64_t lds;
  double* dst;
  int64_t ldd;
  int64_t bs, cols;
  int pr, kv;
  double gv[kMaxGen * kMaxGrid];   // G~_v = [G~_1  V~], K_v x p_r row-major
};

// dA = X_top + G_v^T X_bottom (encoding adjoint), X with m + K_v bs rows.
struct FoldArgs {
  const double* X;
  int64_t ldx;
  double* dA;
  int64_t ldd;
  int64_t m, bs, cols;
  int pr, kv;
  double gv[kMaxGen * kMaxGrid];   // G~_v, K_v x p_r row-major
};

// Scratch regions inside the caller's workspace (all device pointers).
struct Scratch {
  int* info;          // [0]: 0, or 1 + the first panel that is exactly rank-deficient;
                      // [1]: whether the current leaf's first Cholesky pass broke down;
                      // [2]: leaves orthogonalised by the column-wise fallback
  int* fb;            // per panel: 1 if its second pass took the column-wise fallback
  double* part;       // split-K partial tiles
  int64_t npart;      // capacity in tiles (of kTile*kTile doubles)
  double* S;          // projection coefficients (and the fused first-pass Gram)
  double* G;          // Gram matrix and lookahead product (kLeaf x 2 kLeaf)
  double* T;          // inverse Cholesky factor (kLeaf x kLeaf)
  double* R1;         // first-pass Cholesky factor (kLeaf x kLeaf)
  double* X;          // two first-pass panel copies (ldx x b each, xstride doubles apart)
  int64_t ldx, xstride;
  double* T2;         // the second pass's inverse factor, kept for the update stream
  double* colw;       // column-wise panel partial sums (kColWorkDoubles)
};

// Kernel-instance tags: each use of a product kernel gets its own symbol, so
// per-kernel profiles map onto the steps of the factorization.
enum : int { TAG_TRAIL = 0, TAG_REPROJ = 1, TAG_PANEL = 2, TAG_ADJ = 3 };

// C (M x N) = A^T B, A: K x M (lda), B: K x N (ldb), split over K; C2's first M2
// rows += A^T B.  Either of C and C2 may be nullptr.
struct TnArgs {
  const double* A; int64_t lda;
  const double* B; int64_t ldb;
  int M, N; int64_t K;
  int64_t kchunk; int nsplit; int tilesN; int ntiles;
  double* C; int64_t ldc;
  double* C2; int64_t ldc2;
  int M2;             // only rows i < M2 are added into C2
  double* part;
  int vec;            // both operands 16-byte aligned with even leading dimensions
  int f32;            // FP32 products (operands rounded), FP32 sums over 16
                      // k-values, FP64 sums across those groups
  int prio;           // raise the waves' issue priority (panel-chain products)
  int pair;           // two tile rows per 512-thread workgroup (tn2_kernel)
  int quad;           // 128 x 128 output per 512-thread workgroup (tnq_kernel, FP64)
  int bf3;            // split-BF16 product (tnb_kernel): each FP64 operand as hi + mid + lo
                      // BF16 parts, six part products on BF16 MFMA with FP32 sums over
                      // 32 k-values, FP64 sums across them (output layout as f32)
  int seq;            // sum the splits one after the other, in one order for every count
  int lower;          // square product, 128 x 128 blocks above the diagonal left out (quad only)
  int small;          // 16 x 16 outputs per workgroup, the depth shared by its waves (tns_kernel)
};

// Choose the split of C = A^T B (stored to C; rows below M2 -- all rows
// unless changed -- also added into C2 if C2 != nullptr).
// force_split > 0 fixes the split count (capped by the partial capacity).
// lowp: 1 = the product on FP32 MFMA (operands rounded to FP32, FP32 sums over
// 16 k-values, FP64 sums across them); 2 = split BF16 (tnb_kernel) where the
// shape allows it (at least two tile rows and columns, depth a multiple of
// 32, aligned operands), else FP32; for the mixed-precision coefficient
// product R_bar = Qbar^T Q_t.
// fine: splits of fewer than 256 rows where the product is small (split_rows).
TnArgs tn_setup(const double* A, int64_t lda, const double* B, int64_t ldb, int M, int N, int64_t K, double* C,
                int64_t ldc, double* C2, int64_t ldc2, const Scratch& s, int force_split = 0, int lowp = 0,
                bool fine = false);
// C = A^T B (N x N) of which only the lower triangle is read
TnArgs tn_setup_lower(const double* A, int64_t lda, const double* B, int64_t ldb, int N, int64_t K, double* C,
                      int64_t ldc, const Scratch& s);
// Turn a (FP64) into a product on tns_kernel, unsplit, if it is small enough.
bool tn_small(TnArgs& a);
// The product; with nsplit == 1 it stores C (and C2) itself, else partials.
void launch_tn_product(const TnArgs& a, int tag, hipStream_t st);
// Sum the partials into C (and C2) in split order (nsplit > 1 only).
void launch_tn_reduce(const TnArgs& a, hipStream_t st);
// out (w x N, ldo) = T^T W for the product W = A^T B of a (a.M = w <= 64 rows,
// one tile row): W is summed from the split partials (nsplit > 1) or read from
// a.C (nsplit == 1, where the product stored it); T is w x w (ld w).
// fb, P, ldp: when *fb is set (the panel's second pass took the column-wise
// fallback) out = P^T B is formed directly from the finished panel P instead.
void launch_tn_reduce_tmul(const TnArgs& a, const double* T, int w, double* out, int64_t ldo, hipStream_t st,
                           const int* fb = nullptr, const double* P = nullptr, int64_t ldp = 0);

// C (M x N) -= A (M x K) B (K x N).
struct NnArgs {
  double* C; int64_t ldc;
  const double* A; int64_t lda;
  const double* B; int64_t ldb;
  int64_t M; int N; int K;
  int kchunk; int nsplit; int tilesN; int ntiles;
  int vec;            // B 16-byte aligned with even ldb (vector B loads)
  double* part;
  int prio;           // raise the waves' issue priority (panel-chain products)
  int small;          // 16 x 16 elements of C per workgroup (nns_kernel)
  int flush;          // > 0: subtract from C's elements after every `flush` k-values (nn_flush)
  // launch_nn_adj only: C = Cin - sign A B (Cin == nullptr: zero), tri: TRI_* flags
  const double* Cin; int64_t ldcin;
  double sign;
  int tri;
};
// Structure of a product's operands, taken tile by tile: A zero for k < i, B
// zero for k < j or for k > j, only C's lower triangle read.
enum : int { TRI_A_UPPER = 1, TRI_B_LOWER = 2, TRI_B_UPPER = 4, TRI_C_LOWER = 8 };
// The update is FP64 in every precision mode: it is a column operation on the
// encoded matrix and must keep the checksum relations to FP64 rounding.
NnArgs nn_setup(double* C, int64_t ldc, const double* A, int64_t lda, const double* B, int64_t ldb, int64_t M,
                int N, int K, const Scratch& s);
// Turn a into an update by nns_kernel, unsplit, if it is small enough.
bool nn_small(NnArgs& a);
// Have a subtract from C after every `depth` k-values (at least 64), unsplit.
void nn_flush(NnArgs& a, int depth);
void launch_nn_product(const NnArgs& a, int tag, hipStream_t st);
void launch_nn_reduce(const NnArgs& a, hipStream_t st);   // nsplit > 1 only
bool launch_nn_adj(const NnArgs& a, hipStream_t st);

// First Cholesky-QR pass: R1 = chol(W) and T = R1^{-1} (w x w, ld w).
struct CholArgs {
  const double* W; int64_t ldw;     // w x w Gram matrix
  int w, panel;
  double* T; double* R1; int* info;
};

// A panel leaf P (mrows x w, w <= kLeaf) in its two Cholesky-QR passes
// (panel_first_kernel, the sum of its Gram partials, panel_second_kernel).
struct PanelArgs {
  double* P; int64_t ldp; int64_t mrows; int w;
  double* Qn;                       // the next panel (w columns, ld ldp), or nullptr
  // first pass: P <- (P - sum of the split partials) T
  const double* part; int nsplit, ntiles;
  const double* T;                  // or formed from c.W by the kernel itself
  CholArgs c;
  double* X; int64_t ldx;           // second destination of the first pass's panel (or nullptr)
  double* gpart;                    // Gram partials (panel_first_blocks x 2 tiles), or nullptr
  double* G; double* Gn;            // P1^T P1 and P1^T Q_next (ld w)
  // second pass
  double* Rout; double* Rbar; int64_t ldr;   // R_panel = R2 R1; the next panel's coefficients
  double* Tcopy;                    // copy of R2^{-1} (w x w, ld w), or nullptr
  int* fb;                          // set to 1 when the column-wise fallback ran (or nullptr)
};
int panel_first_blocks(int64_t mrows, bool gram);
void launch_panel_first(const PanelArgs& a, bool chol, hipStream_t st);
void launch_panel_reduce(const PanelArgs& a, hipStream_t st);
void launch_panel_second(const PanelArgs& a, hipStream_t st);

// One panel leaf orthogonalised column by column (colstep_kernel,
// colmgs_kernel): the rows are split over up to kColGridMax workgroups, and each
// launch takes one step of the method on every slab, leaving per-workgroup
// partial sums (kColSlots each) that every workgroup of the next launch reduces
// in the same order.
enum : int { COLWISE_CGS2 = 0, COLWISE_ICGS = 1, COLWISE_MGS = 2 };
constexpr int kColGridMax = 128;
constexpr int kColSlots = 132;      // two sets of 64 inner products, four others
// partial sums and state words, two buffers alternating by launch (colstep_kernel:
// kColGridMax x kColSlots and four; colgrid_kernel: 256 x 68, and four in all)
constexpr int64_t kColWorkDoubles = 2 * (256 * (int64_t)68 + 4);
static_assert(kColGridMax * kColSlots <= 256 * 68, "scratch");
struct ColArgs {
  double* P; int64_t ldp; int64_t mrows;
  int w, mode;                      // w <= kLeaf; mode: COLWISE_CGS2 / _ICGS / _MGS
  double eta;                       // ICGS: reorthogonalise when ||p after|| < eta ||p before||
  double* Rout; int64_t ldr;        // the panel's R block (w x w, zeros below the diagonal)
  int* info; int panel;             // a zero column sets info[0] = 1 + panel
  double* work;                     // kColWorkDoubles of scratch
};
void launch_colpanel(const ColArgs& a, hipStream_t st);
void launch_colgrid(const ColArgs& a, hipStream_t st);   // the reduced-precision modes

CholArgs chol_args(const double* W, int64_t ldw, int w, int panel, const Scratch& s);

// The split re-projection update (launch_nn_product with nsplit > 1) with the
// first Cholesky pass described by c run by one extra block of the same
// launch; returns false, launching nothing, when the update does not split.
bool launch_nn_chol(const NnArgs& a, const CholArgs& c, hipStream_t st);

void launch_zero_ints(int* p, int n, hipStream_t st);
void launch_fill_zero(double* p, int64_t ld, int64_t rows, int64_t cols, hipStream_t st);
// checksum rows only (a.kv rows of the code g over a.n columns)
void launch_encode_rows(const EncodeArgs& a, hipStream_t st);
// the whole encoding in one pass: checksum rows (g), columns (gc) and corner
void launch_encode_fused(const EncodeArgs& a, hipStream_t st);
void launch_lines(const LinesArgs& a, hipStream_t st);
void launch_erase(const EraseArgs& a, hipStream_t st);
void launch_postorth(const PostArgs& a, hipStream_t st);
// coded solve: Y = Q^T B (Q m x n), then blocked back substitution with R_1
void launch_gemv_t(const double* Q, int64_t ldq, int64_t m, int n, const double* B, int64_t ldb, int nrhs,
                   double* Y, int64_t ldy, hipStream_t st);
// inverted 64 x 64 diagonal blocks of R; X != nullptr: X (n x nrhs) marked unsolved for launch_trsv_flow
void launch_trinv(const double* R, int64_t ldr, int64_t n, double* T, hipStream_t st, double* X = nullptr,
                  int64_t ldx = 0, int nrhs = 0);
// adjoint helpers
void launch_transpose(const double* src, int64_t lds, double* dst, int64_t ldd, int64_t rows, int64_t cols,
                      double scale, bool upper, hipStream_t st);
void launch_copyltu(double* C, int64_t ldc, int64_t n, hipStream_t st);
// C (rows x cols) = scale U V^T (U rowsu x k: zero rows from rowsu on; upper: zero below the diagonal)
void launch_outer(const double* U, int64_t ldu, const double* V, int64_t ldv, int64_t rowsu, int64_t rows,
                  int64_t cols, int k, double scale, bool upper, double* C, int64_t ldc, hipStream_t st);
void launch_gemv_n(const double* A, int64_t lda, int64_t m, int n, const double* x, int64_t ldx, int nrhs,
                   double* y, int64_t ldy, hipStream_t st);
void launch_fold(const FoldArgs& a, hipStream_t st);
// Y (n x n) = block diagonal of the 64 x 64 tiles of T (tile k at T + 4096 k)
void launch_blockdiag(const double* T, double* Y, int64_t ldy, int64_t n, hipStream_t st);
// dst = src (rows x cols)
void launch_copy(const double* src, int64_t lds, double* dst, int64_t ldd, int64_t rows, int64_t cols, hipStream_t st);
// C *= s (rows x cols)
void launch_scale(double* C, int64_t ldc, int64_t rows, int64_t cols, double s, hipStream_t st);
// one level of the triangular inverse by doubling (h a multiple of 64): for every pair of
// adjacent h-blocks W = R12 T22 (second = false), then T12 = -T11 W (second = true)
void launch_inv_level(const double* R, int64_t ldr, double* Rinv, double* W, int64_t n, int64_t h, bool second,
                      hipStream_t st);
// R X = Y (or R^T X = Y) after launch_trinv(R, ..., T, st, X, ldx, nrhs)
void launch_trsv_flow(const double* R, int64_t ldr, double* T, const double* Y, int64_t ldy, double* X, int64_t ldx,
                      int nrhs, int64_t n, bool trans, hipStream_t st);
// The allocation-free solve's scratch: a file-scope device array of
// kSolveScratchBytes, one copy per device.  *ptr receives the current
// device's copy's address (looked up on the first call on each device).
constexpr size_t kSolveScratchBytes = size_t(32) << 20;
hipError_t solve_scratch(void** ptr);

}  // namespace cqr
