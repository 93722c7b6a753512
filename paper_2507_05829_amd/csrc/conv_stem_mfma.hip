// First layers over RGB images (3 x 3 and 7 x 7 filters, 32 channels or a multiple out) on the
// matrix cores: the forms of the first-layer kernels that take those; conv_stem.hip has the rest.
//
// The reduction axis of such a layer (27 or 147 elements) does not come in 16-byte pieces per tap,
// but a row of the filter is 9 or 21 consecutive elements of an image row. Every filter row is
// therefore padded to whole groups of 16 bytes (2 or 3 of 8 bf16 elements, 3 or 6 of 4 fp32), and two
// groups are one step of the reduction, one for each half of a wavefront: 3 steps for 3 x 3 in bf16,
// 11 for 7 x 7. The padding multiplies zero weights; what a lane read there is cleared first, so
// that an infinite or NaN pixel reaches only the windows it lies in.
//
// A workgroup owns TH output rows x 64 columns and all (or a slice of 32) output channels. The image
// rows under it are staged in LDS once, 4 bytes per load, zero outside the image, starting at the
// first window's first element: a window then starts on a 4-byte boundary (in bf16 with stride 1 every
// second one does: an extra copy, shifted by one element, serves the others). The weights stay in
// registers, and a wavefront takes one 32-pixel fragment at a time from the reads to the stores: sums for one
// fragment leave room for 2 to 7 wavefronts per SIMD (two where 7 x 7 bf16 weights of 64 channels fill the registers; all four fragments of the 8-row form: 2 to 4), whose stores and
// products overlap. Bound by the output it writes. us for the 8-row form, before (whole tile's sums; stores of 32
// bytes per pixel) and now: 3 x 3 stride 2 in bf16, 32 channels, 1080 x 640 outputs 19.0 -> 15.0, 64 channels, stride 1,
// 1150 x 224 16.3 -> 12.9, fp32 3 x 640 x 640 x 64 121 -> 105. 7 x 7 in fp32 is bound by its matrix instructions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>

#include "act.hpp"
#include "conv_common.hpp"
#include "conv_split.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

constexpr int kTileCols = 64;

struct StemMfmaParams {
  const void* x;
  void* y;
  void* y2;           // second destination with y's layout, or nullptr
  const void* w;      // [C_out / 32][step][lane] 16 bytes
  const void* w3;     // fp32 7 x 7: the same as three bf16 parts, [C_out / 32][step of the bf16 form][part][lane] 16 bytes
  const float* bias;  // or nullptr
  int x_row0, x_rows, W;
  int y_row0, y_rows, W_out, C_out;
  int ph, pw, act, out_lo, R, N;
  int tiles_x, tiles_y;
  int conv_h, conv_w;                // pooled form: the convolution's outputs (y, out_lo, R, W_out are the pooling's)
  FastDiv by_x, by_y;
};

template <typename T, int KH> struct StemShape {
  static constexpr int KJ = 3 * KH;                          // elements of a filter row (three channels)
  static constexpr int KE = 16 / (int)sizeof(T);             // elements per group
  static constexpr int G = (KJ + KE - 1) / KE;               // groups per filter row
  static constexpr int STEPS = (KH * G + 1) / 2;
  static constexpr int EPD = 4 / (int)sizeof(T);             // elements per 4-byte word
};

// ROWS image rows from row ih0 and element e0 of a row on into LDS (copy c from the element c further on), zero
// outside the image and the slab: all loads first. NW wavefronts.
template <typename T, int NW, int ROWS, int WORDS, int PITCH, int COPIES>
__device__ __forceinline__ void stem_stage(const StemMfmaParams& p, unsigned (&patch)[COPIES][ROWS * PITCH], int n, int ih0, int e0,
                                           int wave, int lane) {
  constexpr int EPD = 4 / (int)sizeof(T), RPW = (ROWS + NW - 1) / NW, CPL = (WORDS + 63) / 64;
  const int row_elems = p.W * 3;
  unsigned v[COPIES][RPW][CPL];
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int r = wave + NW * i, ih = ih0 + r;
    const bool row_ok = r < ROWS && ih >= p.x_row0 && ih < p.x_row0 + p.x_rows;
    const T* const row = (const T*)p.x + (size_t)(n * p.x_rows + (row_ok ? ih - p.x_row0 : 0)) * row_elems;
#pragma unroll
    for (int c = 0; c < COPIES; ++c)
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        const int e = e0 + (lane + 64 * j) * EPD + c;
        v[c][i][j] = 0u;
        if (row_ok & (e >= 0) & (e + EPD <= row_elems)) {
          __builtin_memcpy(&v[c][i][j], row + e, 4);
        } else if constexpr (EPD == 2) {
          // the word half inside the image
          if (row_ok & (e == -1)) { unsigned short h; __builtin_memcpy(&h, row, 2); v[c][i][j] = (unsigned)h << 16; }
          if (row_ok & (e == row_elems - 1)) { unsigned short h; __builtin_memcpy(&h, row + e, 2); v[c][i][j] = h; }
        }
      }
  }
#pragma unroll
  for (int i = 0; i < RPW; ++i)
#pragma unroll
    for (int c = 0; c < COPIES; ++c)
#pragma unroll
      for (int j = 0; j < CPL; ++j)
        if (wave + NW * i < ROWS && lane + 64 * j < WORDS) patch[c][(wave + NW * i) * PITCH + lane + 64 * j] = v[c][i][j];
}

// The products of 32 windows (win: this lane's) with NT x 32 channels. Group g: filter row g / G, elements (g % G) KE ..;
// step t is groups 2 t (lower half of the wavefront) and 2 t + 1.
template <typename T, int KH, int NT, int PITCH>
__device__ __forceinline__ void stem_products(const unsigned* win, int half, const u32x4 (&w)[StemShape<T, KH>::STEPS][NT], f32x16 (&acc)[NT]) {
  using Sh = StemShape<T, KH>;
  constexpr int KE = Sh::KE, G = Sh::G, STEPS = Sh::STEPS, KJ = Sh::KJ, EPD = Sh::EPD, GROUPS = KH * G;
  // words of the last group of a filter row that hold elements of it
  auto last_mask = [](int j) constexpr {
    const int left = KJ - (G - 1) * KE - j * EPD;
    return left >= EPD ? 0xffffffffu : left <= 0 ? 0u : 0xffffu;
  };
  const unsigned upper = half ? 0xffffffffu : 0u;
#pragma unroll
  for (int t = 0; t < STEPS; ++t) {
    const int ga = 2 * t, gb = 2 * t + 1 < GROUPS ? 2 * t + 1 : 2 * t;
    const int at = (ga / G) * PITCH + (ga % G) * (KE / EPD), bt = (gb / G) * PITCH + (gb % G) * (KE / EPD);
    const unsigned* const src = win + (half ? bt : at);
    u32x4 d = u32x4{src[0], src[1], src[2], src[3]};
    const bool a_last = ga % G == G - 1, b_last = gb % G == G - 1, b_none = 2 * t + 1 >= GROUPS;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned ma = a_last ? last_mask(j) : 0xffffffffu;
      const unsigned mb = b_none ? 0u : b_last ? last_mask(j) : 0xffffffffu;
      if (ma != 0xffffffffu || mb != 0xffffffffu) d[j] &= (mb & upper) | (ma & ~upper);
    }
#pragma unroll
    for (int k = 0; k < NT; ++k) mma<T>(w[t][k], d, acc[k]);
  }
}

template <typename T, int KH, int S, int NT, int TH>
__device__ __forceinline__ void stem_body(const StemMfmaParams& p, const int bx) {
  using Sh = StemShape<T, KH>;
  constexpr int KE = Sh::KE, G = Sh::G, STEPS = Sh::STEPS, EPD = Sh::EPD;
  constexpr int ROWS = (TH - 1) * S + KH;                    // image rows under the tile
  // words of a staged row: the last window's groups end inside it
  constexpr int WORDS = (((kTileCols - 1) * S * 3 + G * KE) + EPD - 1) / EPD + 1;
  constexpr int PITCH = WORDS | 1;                           // (odd: rows start on different banks)
  constexpr int COPIES = sizeof(T) == 2 && S == 1 ? 2 : 1;   // the second starts one element further on
  constexpr int FW = TH / 2;                                 // 32-pixel fragments per wavefront
  __shared__ unsigned patch[COPIES][ROWS * PITCH];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, px = lane & 31;
  const int q = fastdiv(bx, p.by_x), tx = bx - q * p.tiles_x;
  const int n = fastdiv(q, p.by_y), ty = q - n * p.tiles_y;
  const int r0 = ty * TH, c0 = tx * kTileCols;

  stem_stage<T, 4, ROWS, WORDS, PITCH, COPIES>(p, patch, n, (p.out_lo + r0) * S - p.ph, (c0 * S - p.pw) * 3, wave, lane);
  u32x4 w[STEPS][NT];
#pragma unroll
  for (int k = 0; k < NT; ++k)
#pragma unroll
    for (int t = 0; t < STEPS; ++t) w[t][k] = ((const u32x4*)p.w)[((size_t)(blockIdx.y * NT + k) * STEPS + t) * 64 + lane];
  __syncthreads();

  const Clamp cl = make_clamp(p.act);
  T* const yg = (T*)p.y;
  T* const y2 = (T*)p.y2;
  constexpr int PE = 16 / (int)sizeof(T);                    // channels per piece
  const int piece = (lane >> 5) + ((lane >> 4) & 1) * 2;     // of a pixel's four that this lane stores
  f32x4 bias[NT][4];
  auto load_bias = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        bias[k][g] = p.bias ? *(const f32x4*)(p.bias + (blockIdx.y * NT + k) * 32 + g * 8 + half * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
  };
  if constexpr (FW > 1) load_bias();
#pragma unroll 1
  for (int f = 0; f < FW; ++f) {
    const int idx = wave * FW + f, r = idx >> 1, col = (idx & 1) * 32 + px;
    const int e = col * S * 3;                               // first element of the window in a staged row
    f32x16 acc[NT];
#pragma unroll
    for (int a = 0; a < NT; ++a)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][i] = 0.f;
    const unsigned* const win = patch[COPIES == 2 ? (e & 1) : 0] + r * S * PITCH + e / EPD;
    stem_products<T, KH, NT, PITCH>(win, half, w, acc);
    // ---- bias, activation, the one rounding: a lane holds channels 8 g + 4 half + {0..3} of its pixel. Two pieces
    // of 16 bytes of 32 pixels become one store of four pieces of the first 16 pixels and one of the others: a
    // store then writes 64 consecutive bytes of a pixel instead of 32 (19.0 -> 17.4 us on 1080 x 640 x 32).
    if constexpr (FW == 1) load_bias();
    const int row = r0 + r, ocol = c0 + (idx & 1) * 32 + (lane & 15);
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const size_t at = ((size_t)(n * p.y_rows + p.out_lo + row - p.y_row0) * p.W_out + ocol) * p.C_out + (blockIdx.y * NT + k) * 32 + piece * PE;
      float v[16];
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[g * 4 + j] = clamp_act(acc[k][g * 4 + j] + bias[k][g][j], cl);
      auto put = [&](u32x4 a, u32x4 b, int channel) __attribute__((always_inline)) {
        u32x4 lo, hi;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const auto s2 = __builtin_amdgcn_permlane16_swap(a[j], b[j], false, false);
          lo[j] = s2[0]; hi[j] = s2[1];
        }
        if ((row < p.R) & (ocol < p.W_out)) {
          *(u32x4*)(yg + at + channel) = lo;
          if (y2) *(u32x4*)(y2 + at + channel) = lo;
        }
        if ((row < p.R) & (ocol + 16 < p.W_out)) {
          *(u32x4*)(yg + at + (size_t)16 * p.C_out + channel) = hi;
          if (y2) *(u32x4*)(y2 + at + (size_t)16 * p.C_out + channel) = hi;
        }
      };
      if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int g = 0; g < 4; g += 2)
          put(__builtin_bit_cast(u32x4, (f32x4{v[g * 4], v[g * 4 + 1], v[g * 4 + 2], v[g * 4 + 3]})),
              __builtin_bit_cast(u32x4, (f32x4{v[g * 4 + 4], v[g * 4 + 5], v[g * 4 + 6], v[g * 4 + 7]})), g * 8);
      } else {
        // (pieces of 4 + 4 channels exchanged between the halves: 8 consecutive ones per lane)
        u32x4 out[2];
#pragma unroll
        for (int g = 0; g < 4; g += 2) {
          alignas(16) __bf16 o[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) o[j] = (__bf16)v[g * 4 + j];
          const u32x4 b = *(const u32x4*)o;
          const auto s0 = __builtin_amdgcn_permlane32_swap(b[0], b[2], false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(b[1], b[3], false, false);
          out[g / 2] = u32x4{(unsigned)s0[0], (unsigned)s1[0], (unsigned)s0[1], (unsigned)s1[1]};
        }
        put(out[0], out[1], 0);
      }
    }
  }
}

// Small launches: 2 rows per workgroup, so that there are many of them; large ones: 8 rows, which
// stage 1.1 to 1.6 x the rows they need instead of 1.5 to 4.5 x (4 rows measured like 2 on the launches
// between: 7 x 7 fp32 on 640 x 112 pixels 19.7 us against 19.3).
template <typename T, int KJ, int S, int NT>
__global__ __launch_bounds__(256) void conv_stem_mfma_kernel(const StemMfmaParams p) {
  stem_body<T, KJ / 3, S, NT, 2>(p, blockIdx.x);
}
template <typename T, int KJ, int S, int NT>
__global__ __launch_bounds__(256) void conv_stem_mfma_kernel_bands(const Batch<StemMfmaParams> t) {
  const int b = batch_find(t, blockIdx.x);
  stem_body<T, KJ / 3, S, NT, 2>(t.p[b], blockIdx.x - t.first[b]);
}
template <typename T, int KJ, int S, int NT>
__global__ __launch_bounds__(256) void conv_stem_mfma_tall_kernel(const StemMfmaParams p) {
  stem_body<T, KJ / 3, S, NT, 8>(p, blockIdx.x);
}
template <typename T, int KJ, int S, int NT>
__global__ __launch_bounds__(256) void conv_stem_mfma_tall_kernel_bands(const Batch<StemMfmaParams> t) {
  const int b = batch_find(t, blockIdx.x);
  stem_body<T, KJ / 3, S, NT, 8>(t.p[b], blockIdx.x - t.first[b]);
}

// The 7 x 7 stride-2 layer and the 3 x 3 stride-2 max pooling (one row and column of padding) that is its only reader, in
// one launch: a workgroup of eight wavefronts owns 7 x 8 pooled pixels and computes the 15 x 17 outputs of the
// convolution under them, one 32-pixel fragment a wavefront (the 255 fill eight); rounded to the storage type they
// meet in LDS. Neighbouring tiles compute 1.14 times the outputs, for which those need not be written and read
// back, and a chain has one launch less. Four fp32 bands of 224 x 224 into 64 channels: 18.6 + 6.6 us apart, 12.9 here;
// a chain of 21 layers on three bf16 images of 173 x 201 92.4 -> 85.9 us. (With the fp32 instructions such a
// chain of four bands in flight took 129 us instead of 124 apart; with parts 120.)
// fp32 products run on the bf16 matrix cores as sums of three parts (see conv_gemm.hip), 2 100 cycles a
// fragment instead of 5 400: the image is split on its way to LDS, the weights lie there as well (all
// wavefronts need all of them). A wavefront that ends with a sum that is not finite computes its fragment again on the fp32
// instructions (one image of 224 x 224: 7.0 us without such a sum, 15 with one, 19 with one in every fragment). That also covers what is read behind a window's end: an infinity there times the padding's
// zero weight is no finite sum.
constexpr int kPoolRows = 7, kPoolCols = 8;
constexpr int kPoolCR = 2 * kPoolRows + 1, kPoolCC = 2 * kPoolCols + 1;   // outputs of the convolution under a tile
constexpr int kPoolImage = (kPoolCR - 1) * 2 + 7;                          // image rows under those
static_assert(kPoolCR * kPoolCC <= 256, "a fragment per wavefront");
typedef StemShape<__bf16, 7> Stem7;   // the groups and steps of the products in bf16, whole or in parts
constexpr int kPoolWords = ((kPoolCC - 1) * 6 + Stem7::G * 8) / 2, kPoolPitch = kPoolWords | 1;   // of an image row (or part of it) in LDS

// What a tile needs before and after the products: where it lies.
struct StemPoolAt { int n, r0, c0, cr0, cc0; };
__device__ __forceinline__ StemPoolAt stem_pool_at(const StemMfmaParams& p, int bx) {
  const int q = fastdiv(bx, p.by_x), tx = bx - q * p.tiles_x;
  const int n = fastdiv(q, p.by_y), r0 = (q - n * p.tiles_y) * kPoolRows, c0 = tx * kPoolCols;
  return {n, r0, c0, (p.out_lo + r0) * 2 - 1, c0 * 2 - 1};
}

// Bias, activation, the one rounding into LDS (conv: 256 pixels; the caller's barrier lies between its last readers and
// this), and the pooling: 16 bytes of a pooled pixel a thread.
template <typename T, int NT>
__device__ __forceinline__ void stem_pool_finish(const StemMfmaParams& p, unsigned char* conv, const f32x16 (&acc)[NT], const StemPoolAt& t,
                                                 int cr, int cc, int px, int half) {
  constexpr int OUT = NT * 32 * (int)sizeof(T), OUT_PITCH = OUT + 16;   // bytes of a pixel
  const Clamp cl = make_clamp(p.act);
  // (an output outside the image is no part of a maximum)
  const bool inside = (t.cr0 + cr >= 0) & (t.cr0 + cr < p.conv_h) & (t.cc0 + cc >= 0) & (t.cc0 + cc < p.conv_w);
#pragma unroll
  for (int k = 0; k < NT; ++k)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int c = k * 32 + g * 8 + half * 4;
      const f32x4 bias = p.bias ? *(const f32x4*)(p.bias + blockIdx.y * (NT * 32) + c) : f32x4{0.f, 0.f, 0.f, 0.f};
      alignas(16) T o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = from_f32<T>(inside ? clamp_act(acc[k][g * 4 + j] + bias[j], cl) : -INFINITY);
      __builtin_memcpy(__builtin_assume_aligned(conv + px * OUT_PITCH + c * sizeof(T), 4 * sizeof(T)), o, sizeof(o));
    }
  __syncthreads();

  constexpr int PIECES = OUT / 16, VE = 16 / (int)sizeof(T);
  const int piece = threadIdx.x % PIECES, pp = threadIdx.x / PIECES, pr = pp / kPoolCols, pc = pp - pr * kPoolCols;
  if (pr >= kPoolRows || t.r0 + pr >= p.R || t.c0 + pc >= p.W_out) return;
  float best[VE];
#pragma unroll
  for (int j = 0; j < VE; ++j) best[j] = -INFINITY;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      alignas(16) T v[VE];
      *(u32x4*)v = *(const u32x4*)(conv + ((2 * pr + a) * kPoolCC + 2 * pc + b) * OUT_PITCH + piece * 16);
#pragma unroll
      for (int j = 0; j < VE; ++j) best[j] = fmaxf(best[j], to_f32(v[j]));
    }
  alignas(16) T o[VE];
#pragma unroll
  for (int j = 0; j < VE; ++j) o[j] = from_f32<T>(best[j]);
  const size_t to =
      ((size_t)(t.n * p.y_rows + p.out_lo + t.r0 + pr - p.y_row0) * p.W_out + t.c0 + pc) * p.C_out + blockIdx.y * (NT * 32) + piece * VE;
  *(u32x4*)((T*)p.y + to) = *(const u32x4*)o;
  if (p.y2) *(u32x4*)((T*)p.y2 + to) = *(const u32x4*)o;
}

template <int NT>
__device__ __forceinline__ void stem_pool_body(const StemMfmaParams& p, const int bx) {
  constexpr int STEPS = Stem7::STEPS;
  __shared__ unsigned patch[1][kPoolImage * kPoolPitch];
  __shared__ __attribute__((aligned(16))) unsigned char conv[256 * (NT * 64 + 16)];
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const StemPoolAt t = stem_pool_at(p, bx);
  stem_stage<__bf16, 8, kPoolImage, kPoolWords, kPoolPitch, 1>(p, patch, t.n, t.cr0 * 2 - p.ph, (t.cc0 * 2 - p.pw) * 3, wave, lane);
  u32x4 w[STEPS][NT];
#pragma unroll
  for (int k = 0; k < NT; ++k)
#pragma unroll
    for (int s = 0; s < STEPS; ++s) w[s][k] = ((const u32x4*)p.w)[((size_t)(blockIdx.y * NT + k) * STEPS + s) * 64 + lane];
  __syncthreads();

  const int px = wave * 32 + (lane & 31), at = min(px, kPoolCR * kPoolCC - 1), cr = at / kPoolCC, cc = at - cr * kPoolCC;
  f32x16 acc[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[k][i] = 0.f;
  stem_products<__bf16, 7, NT, kPoolPitch>(patch[0] + cr * 2 * kPoolPitch + cc * 3, half, w, acc);
  stem_pool_finish<__bf16, NT>(p, conv, acc, t, cr, cc, px, half);
}

__device__ __forceinline__ void stem_pool_split_body(const StemMfmaParams& p, const int bx) {
  constexpr int STEPS = Stem7::STEPS, G = Stem7::G, GROUPS = 7 * G;
  constexpr int IMAGE = 3 * kPoolImage * kPoolPitch;        // words: [part][row][word]
  constexpr int WPIECES = STEPS * 3 * 64, WPT = (WPIECES + 511) / 512;
  constexpr int W_BYTES = WPIECES * 16, CONV = 256 * (128 + 16);
  constexpr int SMEM = W_BYTES + IMAGE * 4 > CONV ? W_BYTES + IMAGE * 4 : CONV;
  __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];
  u32x4* const ws = (u32x4*)smem;
  unsigned* const image = (unsigned*)(smem + W_BYTES);
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const StemPoolAt t = stem_pool_at(p, bx);

  // ---- the image, two elements a word and part, and the weights: all loads first
  const int ih0 = t.cr0 * 2 - p.ph, e0 = (t.cc0 * 2 - p.pw) * 3, row_elems = p.W * 3;
  constexpr int RPW = (kPoolImage + 7) / 8;
  static_assert(kPoolWords <= 64, "a lane per word of a row");
  float v[RPW][2];
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int r = wave + 8 * i, ih = ih0 + r, e = e0 + lane * 2;
    const bool row_ok = r < kPoolImage && ih >= p.x_row0 && ih < p.x_row0 + p.x_rows;
    const float* const row = (const float*)p.x + (size_t)(t.n * p.x_rows + (row_ok ? ih - p.x_row0 : 0)) * row_elems;
    v[i][0] = v[i][1] = 0.f;
    if (row_ok & (e >= 0) & (e < row_elems)) v[i][0] = row[e];
    if (row_ok & (e + 1 >= 0) & (e + 1 < row_elems)) v[i][1] = row[e + 1];
  }
  u32x4 wv[WPT];
  const u32x4* const w3 = (const u32x4*)p.w3 + (size_t)blockIdx.y * WPIECES;
#pragma unroll
  for (int i = 0; i < WPT; ++i) wv[i] = w3[min(tid + i * 512, WPIECES - 1)];
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    unsigned parts[3];
    split_bf16(v[i][0], v[i][1], parts);
    if (wave + 8 * i < kPoolImage && lane < kPoolWords) {
#pragma unroll
      for (int k = 0; k < 3; ++k) image[(k * kPoolImage + wave + 8 * i) * kPoolPitch + lane] = parts[k];
    }
  }
#pragma unroll
  for (int i = 0; i < WPT; ++i)
    if (tid + i * 512 < WPIECES) ws[tid + i * 512] = wv[i];
  __syncthreads();

  // ---- the products, step by step as in stem_products
  const int px = wave * 32 + (lane & 31), at = min(px, kPoolCR * kPoolCC - 1), cr = at / kPoolCC, cc = at - cr * kPoolCC;
  f32x16 acc[1][1], low[1][1];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[0][0][i] = low[0][0][i] = 0.f;
  const unsigned* const win = image + cr * 2 * kPoolPitch + cc * 3;
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int ga = 2 * s, gb = 2 * s + 1 < GROUPS ? 2 * s + 1 : 2 * s;   // (the last step's second group: zero weights)
    const unsigned* const src = win + (half ? (gb / G) * kPoolPitch + (gb % G) * 4 : (ga / G) * kPoolPitch + (ga % G) * 4);
    u32x4 w[1][3], x[1][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const unsigned* const sk = src + k * (kPoolImage * kPoolPitch);
      x[0][k] = u32x4{sk[0], sk[1], sk[2], sk[3]};
      w[0][k] = ws[(s * 3 + k) * 64 + lane];
    }
#pragma unroll
    for (int e = 0; e < 6; ++e) mma_split_part<1, 1>(w, x, acc, low, e);
  }
  f32x16 sum[1];
  sum[0] = (acc[0][0] + low[0][0]) * kSplitUnscale;
  float odd = 0.f;   // NaN if a sum is not finite
#pragma unroll
  for (int i = 0; i < 16; ++i) odd += sum[0][i] - sum[0][i];
  if (__builtin_amdgcn_ballot_w64(!(odd == 0.f))) {
    typedef StemShape<float, 7> F;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[0][i] = 0.f;
    for (int s = 0; s < F::STEPS; ++s) {
      const int g = 2 * s + half, a = g / F::G, j0 = g % F::G * 4;   // filter row, first element of it
      const int ih = ih0 + cr * 2 + a, e = e0 + cc * 6 + j0;
      const bool row_ok = a < 7 && ih >= p.x_row0 && ih < p.x_row0 + p.x_rows;
      f32x4 d = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (row_ok & (j0 + j < F::KJ) & (e + j >= 0) & (e + j < row_elems))
          d[j] = ((const float*)p.x)[(size_t)(t.n * p.x_rows + ih - p.x_row0) * row_elems + e + j];
      mma<float>(((const u32x4*)p.w)[((size_t)blockIdx.y * F::STEPS + s) * 64 + lane], __builtin_bit_cast(u32x4, d), sum[0]);
    }
  }
  __syncthreads();   // (the outputs go where the image and the weights were)
  stem_pool_finish<float, 1>(p, smem, sum, t, cr, cc, px, half);
}

// (NT: tiles of 32 channels a wavefront; one in fp32)
template <typename T, int NT>
__device__ __forceinline__ void stem_pool(const StemMfmaParams& p, const int bx) {
  if constexpr (sizeof(T) == 4) stem_pool_split_body(p, bx);
  else stem_pool_body<NT>(p, bx);
}
template <typename T, int NT>
__global__ __launch_bounds__(512) void conv_stem_pool_kernel(const StemMfmaParams p) {
  stem_pool<T, NT>(p, blockIdx.x);
}
template <typename T, int NT>
__global__ __launch_bounds__(512) void conv_stem_pool_kernel_bands(const Batch<StemMfmaParams> t) {
  const int b = batch_find(t, blockIdx.x);
  stem_pool<T, NT>(t.p[b], blockIdx.x - t.first[b]);
}

// Bytes of the packing for the matrix cores, and of the three parts behind it (the pooled form's in fp32).
size_t stem_mfma_whole_bytes(int c_out, int kh, int dtype) {
  const int steps = dtype == LOP_BF16 ? (kh == 3 ? StemShape<__bf16, 3>::STEPS : StemShape<__bf16, 7>::STEPS)
                                      : (kh == 3 ? StemShape<float, 3>::STEPS : StemShape<float, 7>::STEPS);
  return (size_t)(c_out / 32) * steps * 64 * 16;
}
size_t stem_mfma_parts_bytes(int c_out, int kh, int dtype) { return dtype == LOP_BF16 || kh != 7 ? 0 : (size_t)(c_out / 32) * Stem7::STEPS * 3 * 64 * 16; }

StemMfmaParams make_stem_mfma(const OpLaunch& L) {
  StemMfmaParams p = {};
  p.x = L.x.ptr; p.y = L.y.ptr; p.y2 = L.y2; p.bias = L.bias;
  p.w = (const char*)L.wstem + stem_mfma_offset(L.x.c, L.y.c, L.kh, L.kw);
  p.w3 = (const char*)p.w + stem_mfma_whole_bytes(L.y.c, L.kh, L.dtype);
  p.x_row0 = L.x.row0; p.x_rows = L.x.rows; p.W = L.x.w;
  p.y_row0 = L.y.row0; p.y_rows = L.y.rows; p.W_out = L.y.w; p.C_out = L.y.c;
  p.ph = L.ph; p.pw = L.pw; p.act = L.act; p.out_lo = L.out_lo; p.R = L.out_hi - L.out_lo; p.N = L.x.n;
  return p;
}
void stem_tiles(StemMfmaParams& p, int rows, int cols) {
  p.tiles_x = (p.W_out + cols - 1) / cols;
  p.tiles_y = (p.R + rows - 1) / rows;
  p.by_x = make_fastdiv(p.tiles_x); p.by_y = make_fastdiv(p.tiles_y);
}

template <typename T, int KH, int S, int NT>
hipError_t launch_form(const OpLaunch* Ls, int n, bool large, hipStream_t s, KernelEvents* ev) {
  StemMfmaParams ps[kMaxBatch];
  unsigned gx[kMaxBatch];
  int m = 0;
  const int th = large ? 8 : 2;
  for (int b = 0; b < n; ++b) {
    StemMfmaParams p = make_stem_mfma(Ls[b]);
    if (p.R <= 0 || p.N <= 0) continue;
    stem_tiles(p, th, kTileCols);
    ps[m] = p;
    gx[m++] = (unsigned)((long)p.N * p.tiles_y * p.tiles_x);
  }
  if (m == 0) return hipSuccess;
  const unsigned gy = (unsigned)(Ls[0].y.c / (32 * NT));
  if (large)
    return launch_group(conv_stem_mfma_tall_kernel<T, 3 * KH, S, NT>, conv_stem_mfma_tall_kernel_bands<T, 3 * KH, S, NT>, ps, m, gx, gy, 1, dim3(256), s, ev);
  return launch_group(conv_stem_mfma_kernel<T, 3 * KH, S, NT>, conv_stem_mfma_kernel_bands<T, 3 * KH, S, NT>, ps, m, gx, gy, 1, dim3(256), s, ev);
}

// 32-channel tiles per wavefront: the filter has to fit in registers (7 x 7 in fp32 is 84 per tile)
int stem_nt(const OpLaunch& L) { return L.y.c % 64 == 0 && !(L.kh == 7 && L.dtype == LOP_F32) ? 2 : 1; }

template <typename T, int KH, int S>
hipError_t launch_nt(const OpLaunch* Ls, int n, bool large, hipStream_t s, KernelEvents* ev) {
  if constexpr (!(KH == 7 && sizeof(T) == 4))
    if (stem_nt(Ls[0]) == 2) return launch_form<T, KH, S, 2>(Ls, n, large, s, ev);
  return launch_form<T, KH, S, 1>(Ls, n, large, s, ev);
}

template <typename T>
hipError_t launch_type(const OpLaunch* Ls, int n, bool large, hipStream_t s, KernelEvents* ev) {
  if (Ls[0].kh == 3) return Ls[0].sh == 1 ? launch_nt<T, 3, 1>(Ls, n, large, s, ev) : launch_nt<T, 3, 2>(Ls, n, large, s, ev);
  return Ls[0].sh == 1 ? launch_nt<T, 7, 1>(Ls, n, large, s, ev) : launch_nt<T, 7, 2>(Ls, n, large, s, ev);
}

template <typename T, int KH>
void pack(const unsigned char* src, int row_pitch, int c_out, unsigned char* dst) {
  using Sh = StemShape<T, KH>;
  for (int co = 0; co < c_out; ++co)
    for (int g = 0; g < KH * Sh::G; ++g)
      for (int j = 0; j < Sh::KE; ++j) {
        const int e = g % Sh::G * Sh::KE + j;
        if (e >= Sh::KJ) continue;
        const size_t at = (((size_t)(co / 32) * Sh::STEPS + g / 2) * 64 + (g % 2) * 32 + co % 32) * Sh::KE + j;
        std::memcpy(dst + at * sizeof(T), src + ((size_t)co * row_pitch + (g / Sh::G) * Sh::KJ + e) * sizeof(T), sizeof(T));
      }
}

// The 7 x 7 fp32 weights as three bf16 parts each (as split_bf16 does it), in the groups and steps of the bf16 form.
void pack_parts(const unsigned char* src, int row_pitch, int c_out, unsigned char* dst) {
  for (int co = 0; co < c_out; ++co)
    for (int g = 0; g < 7 * Stem7::G; ++g)
      for (int j = 0; j < 8; ++j) {
        const int e = g % Stem7::G * 8 + j;
        if (e >= Stem7::KJ) continue;
        float v;
        std::memcpy(&v, src + ((size_t)co * row_pitch + (g / Stem7::G) * Stem7::KJ + e) * 4, 4);
        v *= kSplitScale;
        for (int k = 0; k < 3; ++k) {
          unsigned u;
          std::memcpy(&u, &v, 4);
          const unsigned short part = v != v ? 0x7fc0 : (unsigned short)((u + 0x7fff + ((u >> 16) & 1)) >> 16);
          const size_t at = ((((size_t)(co / 32) * Stem7::STEPS + g / 2) * 3 + k) * 64 + (g % 2) * 32 + co % 32) * 8 + j;
          std::memcpy(dst + at * 2, &part, 2);
          const unsigned w = (unsigned)part << 16;
          float high;
          std::memcpy(&high, &w, 4);
          v -= high;
        }
      }
}

template <typename T, int NT>
hipError_t launch_pool_form(const OpLaunch* convs, const OpLaunch* pools, int n, hipStream_t s, KernelEvents* ev) {
  StemMfmaParams ps[kMaxBatch];
  unsigned gx[kMaxBatch];
  int m = 0;
  for (int b = 0; b < n; ++b) {
    OpLaunch L = convs[b];
    L.y = pools[b].y; L.y2 = pools[b].y2; L.out_lo = pools[b].out_lo; L.out_hi = pools[b].out_hi;
    StemMfmaParams p = make_stem_mfma(L);
    if (p.R <= 0 || p.N <= 0) continue;
    p.conv_h = convs[b].y.h; p.conv_w = convs[b].y.w;
    stem_tiles(p, kPoolRows, kPoolCols);
    ps[m] = p;
    gx[m++] = (unsigned)((long)p.N * p.tiles_y * p.tiles_x);
  }
  if (m == 0) return hipSuccess;
  return launch_group(conv_stem_pool_kernel<T, NT>, conv_stem_pool_kernel_bands<T, NT>, ps, m, gx, (unsigned)(convs[0].y.c / (32 * NT)), 1,
                      dim3(512), s, ev);
}

}  // namespace

bool stem_mfma_shape(int c_in, int c_out, int kh, int kw) { return c_in == 3 && c_out % 32 == 0 && kh == kw && (kh == 3 || kh == 7); }

size_t stem_mfma_offset(int c_in, int c_out, int kh, int kw) { return 2 * (size_t)c_out * c_in * kh * kw * sizeof(float); }

size_t stem_mfma_bytes(int c_out, int kh, int dtype) { return stem_mfma_whole_bytes(c_out, kh, dtype) + stem_mfma_parts_bytes(c_out, kh, dtype); }

// src: the packed rows [c_out][row_pitch], k = (a * kw + b) * 3 + ci, in the storage type
void stem_mfma_pack(const unsigned char* src, int row_pitch, int c_out, int kh, int dtype, unsigned char* dst) {
  if (dtype == LOP_BF16) kh == 3 ? pack<__bf16, 3>(src, row_pitch, c_out, dst) : pack<__bf16, 7>(src, row_pitch, c_out, dst);
  else kh == 3 ? pack<float, 3>(src, row_pitch, c_out, dst) : pack<float, 7>(src, row_pitch, c_out, dst);
  if (stem_mfma_parts_bytes(c_out, kh, dtype)) pack_parts(src, row_pitch, c_out, dst + stem_mfma_whole_bytes(c_out, kh, dtype));
}

bool stem_mfma_applies(const OpLaunch& L) {
  return stem_mfma_shape(L.x.c, L.y.c, L.kh, L.kw) && L.sh == L.sw && (L.sh == 1 || L.sh == 2);
}

hipError_t launch_stem_mfma(const OpLaunch* Ls, int n, bool large, hipStream_t s, KernelEvents* ev) {
  return Ls[0].dtype == LOP_BF16 ? launch_type<__bf16>(Ls, n, large, s, ev) : launch_type<float>(Ls, n, large, s, ev);
}

void stem_mfma_describe(const OpLaunch& L, bool large, const char* form, char* name, size_t size) {
  snprintf(name, size, "conv_stem_mfma_%skernel%s<%s, %d, %d, %d>", large ? "tall_" : "", form, L.dtype == LOP_BF16 ? "__bf16" : "float",
           3 * L.kh, L.sh, stem_nt(L));
}

// Whether the convolution and the max pooling that reads it are one launch of the pooled form.
bool stem_pool_applies(const OpLaunch& conv, const OpLaunch& pool) {
  if (!stem_applies(conv) || !stem_mfma_applies(conv) || conv.kh != 7 || conv.sh != 2) return false;
  return pool.op == LOP_MAXPOOL2D && pool.kh == 3 && pool.kw == 3 && pool.sh == 2 && pool.sw == 2 && pool.ph == 1 && pool.pw == 1 &&
         pool.dh == 1 && pool.dw == 1;
}

hipError_t launch_stem_pool(const OpLaunch* convs, const OpLaunch* pools, int n, hipStream_t s, KernelEvents* ev) {
  if (n < 1 || n > kMaxBatch) return hipErrorInvalidValue;
  for (int b = 0; b < n; ++b)
    if (!stem_pool_applies(convs[b], pools[b])) return hipErrorInvalidValue;
  if (convs[0].dtype != LOP_BF16) return launch_pool_form<float, 1>(convs, pools, n, s, ev);
  return stem_nt(convs[0]) == 2 ? launch_pool_form<__bf16, 2>(convs, pools, n, s, ev) : launch_pool_form<__bf16, 1>(convs, pools, n, s, ev);
}

void stem_pool_describe(const OpLaunch& conv, const char* form, char* name, size_t size) {
  snprintf(name, size, "conv_stem_pool_kernel%s<%s, %d>", form, conv.dtype == LOP_BF16 ? "__bf16" : "float", stem_nt(conv));
}

}  // namespace lop
