// FP64 MFMA primitives shared by the kernels: the 16 x 16 x 4 instruction and
// a 16 x 16 block product over LDS-resident operands (the operand layout is
// described at the head of cqr_gemm.hip).
#pragma once
#include "cqr_kernels.hpp"

namespace cqr {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v4d mfma(double x, double y, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
}

// 16 x 16 block product on MFMA: acc += sum over k < 16 nk of A(i, k) B(k, j)
// for the block's i, j < 16.  Lane (li, g) feeds A(li, k) and B(k, li) for
// k = k0 + 4g + s, and holds C[li][4r + g] in acc[r] (the layout used
// throughout).
template <class FA, class FB>
__device__ __forceinline__ void mma16(v4d& acc, int lane, int nk, FA A, FB B) {
  const int li = lane & 15, g = lane >> 4;
  for (int k0 = 0; k0 < 16 * nk; k0 += 16) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + 4 * g + s;
      acc = mfma(B(k, li), A(li, k), acc);
    }
  }
}

}  // namespace cqr
