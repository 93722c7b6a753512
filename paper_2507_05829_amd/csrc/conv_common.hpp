// Pieces the dense convolution kernels share: operand vectors and matrix products, division by
// numbers only the host knows, and the order in which workgroups take tiles.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.hpp"

namespace lop {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// 16 bytes in registers: a native vector, so that copies of it are loads and stores the
// optimiser can keep in registers (copies of HIP's uint4 struct are memcpy calls, and an
// array of them that is filled from memory stays in private memory)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Division of a pixel index by a width or a row count that only the host knows: q = (mulhi(n,
// mul) + n) >> shift for 0 <= n < 2^31 (Granlund and Montgomery's division by an invariant
// integer), three instructions where the integer division of two registers takes about forty,
// and a wavefront issues one instruction in four cycles or more.
struct FastDiv { unsigned mul; int shift; };
inline FastDiv make_fastdiv(int d) {
  FastDiv f{1u, 0};
  if (d < 1) return f;
  while ((1L << f.shift) < d) ++f.shift;
  f.mul = (unsigned)((((unsigned long long)1 << 32) * (((unsigned long long)1 << f.shift) - (unsigned long long)d)) / (unsigned long long)d + 1);
  return f;
}
__device__ __forceinline__ int fastdiv(int n, const FastDiv& f) {
  return (int)((__umulhi((unsigned)n, f.mul) + (unsigned)n) >> f.shift);
}

// n / d for n < 2^12 and n d < 2^20 (pixels of a tile or a patch) with mul = small_div(d): two instructions at full
// rate, where a product of 32 bits takes four times as long as others.
constexpr unsigned small_div(int d) { return d < 1 ? 0u : ((1u << 20) + (unsigned)d - 1) / (unsigned)d; }
__device__ __forceinline__ int smalldiv(int n, unsigned mul) { return (int)(__umul24((unsigned)n, mul) >> 20); }

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(__bf16 v) { return (float)v; }

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ __bf16 from_f32<__bf16>(float v) { return (__bf16)v; }

template <typename T>
__device__ __forceinline__ void mma(const u32x4& wa, const u32x4& px, f32x16& acc);

template <>
__device__ __forceinline__ void mma<__bf16>(const u32x4& wa, const u32x4& px, f32x16& acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wa),
                                                __builtin_bit_cast(bf16x8, px), acc, 0, 0, 0);
}

template <>
__device__ __forceinline__ void mma<float>(const u32x4& wa, const u32x4& px, f32x16& acc) {
  const f32x4 a = __builtin_bit_cast(f32x4, wa), b = __builtin_bit_cast(f32x4, px);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0], b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[1], b[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[2], b[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[3], b[3], acc, 0, 0, 0);
}

// v + bias, and of each of the four values the maximum over four neighbouring lanes, in all four lanes: the 2 x 2 pooling of
// pixels that lanes hold window by window. Two instructions a value; fmaxf of a moved value is seven, most of them to quiet
// NaNs that a matrix instruction does not make. (An instruction that reads another lane needs two others between it and
// the one that wrote the value, and many more behind a matrix instruction, whose results the compiler does not know to be read
// here: the addition is the vector instruction that lies between in any case.)
__device__ __forceinline__ void max_of_quad(f32x4& v, const f32x4& bias) {
  v += bias;
  float a = v[0], b = v[1], c = v[2], d = v[3];
  asm volatile("s_nop 1\n"
               "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
               "v_max_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
               "v_max_f32_dpp %2, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
               "v_max_f32_dpp %3, %3, %3 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
               "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n"
               "v_max_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n"
               "v_max_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n"
               "v_max_f32_dpp %3, %3, %3 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
               : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
  v = f32x4{a, b, c, d};
}

// The matrix instructions of one operand pair (bf16: one, fp32: four), one at a time: a loop over
// several accumulators issues each accumulator's next one only after the others' current ones, so none
// waits for the result of the one before it.
template <typename T> constexpr int kMmaParts = sizeof(T) == 4 ? 4 : 1;
template <typename T>
__device__ __forceinline__ void mma_part(const u32x4& wa, const u32x4& px, f32x16& acc, int e) {
  if constexpr (sizeof(T) == 2) {
    mma<T>(wa, px, acc);
  } else {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(f32x4, wa)[e], __builtin_bit_cast(f32x4, px)[e], acc, 0, 0, 0);
  }
}

// Which tile a workgroup takes. The hardware hands workgroups to the 8 XCDs round-robin in
// launch order (x fastest), and every XCD has an L2 of its own: in launch order the 64
// workgroups that are resident on one XCD at a time would be scattered over the whole grid
// and each would pull its own pixel tile and weight tile through that L2. Instead XCD k takes
// the k-th contiguous eighth of a walk over the tiles that goes down groups of kGroupM pixel
// tiles and then across the channel tiles, so its resident workgroups form a block of about
// 8 x 8 tiles that shares 8 pixel tiles and 8 weight tiles. Reduction slices are outermost.
struct TileId { int m, n, z; };
constexpr int kXcds = 8, kGroupM = 8;
// (by_group: division by kGroupM * ny, made on the host. The last group of a launch has fewer pixel tiles, and small launches
// have no other: in_group < 8 * 65 535 divided by 1 .. 8 as a product of floats, whose error of 2 in 2^23 parts is less
// than the 1 / 16 that separates (in_group + 1/2) / gm from the next integer.)
__device__ __forceinline__ TileId xcd_tile_of(int launch, int mx, int ny, int nz, const FastDiv& by_group) {
  const int total = mx * ny * nz;
  const int xcd = (unsigned)launch % kXcds, slot = (unsigned)launch / kXcds;
  const int q = (unsigned)total / kXcds, r = (unsigned)total % kXcds;
  const int v = xcd * q + min(xcd, r) + slot;  // XCD k owns q (+1 for the first r) consecutive tiles
  int z = 0, t = v;
  if (nz > 1) {
    const int per_z = mx * ny;
    z = v / per_z;
    t = v - z * per_z;
  }
  const int group = fastdiv(t, by_group), in_group = t - group * (kGroupM * ny);
  const int first = group * kGroupM;
  const int gm = min(kGroupM, mx - first);
  TileId id;
  id.z = z;
  id.n = __builtin_amdgcn_readfirstlane((int)(((float)in_group + 0.5f) * __builtin_amdgcn_rcpf((float)gm)));
  id.m = first + in_group - id.n * gm;
  return id;
}

__device__ __forceinline__ TileId xcd_tile(int bx, int mx, int ny, int nz, const FastDiv& by_group) {
  return xcd_tile_of(bx + mx * (blockIdx.y + ny * blockIdx.z), mx, ny, nz, by_group);
}

// f(integral_constant<0>) ... f(integral_constant<N - 1>): loops whose body needs its index as a constant
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unroll(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll<N, I + 1>(f);
  }
}
// s_waitcnt immediate that waits until at most n vector-memory operations are outstanding
// and leaves the other counters alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14).
constexpr int vmcnt_imm(int n) { return (n & 0xf) | ((n >> 4) << 14) | (0x7 << 4) | (0xf << 8); }


}  // namespace
}  // namespace lop
