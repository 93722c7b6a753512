// fp32 values as sums of three bf16 values, for products on the bf16 matrix cores (conv_gemm.hip says why and
// how precise).
#pragma once
#include <hip/hip_runtime.h>

#include "conv_common.hpp"

namespace lop {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Both operands are multiplied by 2^24 before they are split, and sums of products by 2^-48: exact, and the last bit of
// every part of any fp32 value, subnormal ones included, is then a normal bf16 value (2^-149 becomes 2^-125). Unscaled, the third part of a
// value below 2^-110 would fall under bf16's smallest step, then the second. Operands from 2^104 on and sums from 2^80 on
// become infinite for it; a sum that is not finite is computed again on the fp32 instructions in any case.
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

// 2^24 v = high + middle + low, each rounded to nearest: the remainder of a rounding to 8 bits is exact in fp32, and
// what is left for the third part has at most 8 bits. Two values at a time: one conversion rounds both, and the
// halves of its result are the values to subtract.
__device__ __forceinline__ void split_bf16(float a, float b, unsigned (&parts)[3]) {
  a *= kSplitScale;
  b *= kSplitScale;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    parts[k] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
    if (k < 2) {
      a -= __builtin_bit_cast(float, parts[k] << 16);
      b -= __builtin_bit_cast(float, parts[k] & 0xffff0000u);
    }
  }
}
__device__ __forceinline__ void split_bf16(const f32x4& v, uint2 (&parts)[3]) {
  unsigned lo[3], hi[3];
  split_bf16(v[0], v[1], lo);
  split_bf16(v[2], v[3], hi);
#pragma unroll
  for (int k = 0; k < 3; ++k) parts[k] = make_uint2(lo[k], hi[k]);
}

// The same for the eight values of a matrix operand.
__device__ __forceinline__ void split_bf16(const u32x4& a, const u32x4& b, u32x4 (&parts)[3]) {
  uint2 lo[3], hi[3];
  split_bf16(__builtin_bit_cast(f32x4, a), lo);
  split_bf16(__builtin_bit_cast(f32x4, b), hi);
#pragma unroll
  for (int k = 0; k < 3; ++k) parts[k] = u32x4{lo[k].x, lo[k].y, hi[k].x, hi[k].y};
}

// Whether one of a wavefront's sums is not finite.
template <int N>
__device__ __forceinline__ bool any_not_finite(const f32x16 (&sum)[N]) {
  float odd = 0.f;   // NaN if a sum is not finite
#pragma unroll
  for (int k = 0; k < N; ++k)
#pragma unroll
    for (int i = 0; i < 16; ++i) odd += sum[k][i] - sum[k][i];
  return __builtin_amdgcn_ballot_w64(!(odd == 0.f)) != 0;
}

// The partial products of one operand pair: e = 0 .. 4 the five small ones (for a sum of their own), 5 high x high. Dropped are
// middle x low, low x middle and low x low: |middle| <= 2^-8 and |low| <= 2^-17 of a value, so 2^-24 of the product at most.
constexpr int kSplitW[6] = {2, 0, 1, 1, 0, 0}, kSplitX[6] = {0, 2, 1, 0, 1, 0};

// Partial product e = 0 .. 5 of one step of 16 of the reduction: the five small ones into `low`, high x high into acc.
template <int TN, int TM>
__device__ __forceinline__ void mma_split_part(const u32x4 (&w)[TN][3], const u32x4 (&x)[TM][3], f32x16 (&acc)[TN][TM], f32x16 (&low)[TN][TM],
                                               int e) {
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) mma<__bf16>(w[a][kSplitW[e]], x[b][kSplitX[e]], e < 5 ? low[a][b] : acc[a][b]);
}

}  // namespace
}  // namespace lop
