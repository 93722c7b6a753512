// fp32 values as sums of three bf16 values, for products on the bf16 matrix cores (conv_gemm.hip says why and
// how precise).
#pragma once
#include <hip/hip_runtime.h>

#include "conv_common.hpp"

namespace lop {
namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// v = high + middle + low, each rounded to nearest: the remainder of a rounding to 8 bits is exact in fp32, and
// what is left for the third part has at most 8 bits.
__device__ __forceinline__ void split_bf16(const f32x4& v, uint2 (&parts)[3]) {
  f32x4 left = v;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const bf16x4 b = __builtin_convertvector(left, bf16x4);
    parts[k] = __builtin_bit_cast(uint2, b);
    if (k < 2) left -= __builtin_convertvector(b, f32x4);
  }
}

// Partial product e = 0 .. 5 of one step of 16 of the reduction: the five small ones into `low`, high x high into acc.
template <int TN, int TM>
__device__ __forceinline__ void mma_split_part(const u32x4 (&w)[TN][3], const u32x4 (&x)[TM][3], f32x16 (&acc)[TN][TM], f32x16 (&low)[TN][TM],
                                               int e) {
  constexpr int kW[6] = {2, 0, 1, 1, 0, 0}, kX[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) mma<__bf16>(w[a][kW[e]], x[b][kX[e]], e < 5 ? low[a][b] : acc[a][b]);
}

}  // namespace
}  // namespace lop
