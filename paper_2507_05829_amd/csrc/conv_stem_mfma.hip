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
// fragment leave room for 3 to 7 wavefronts per SIMD (all four fragments of the 8-row form: 2 to 4), whose stores and
// products overlap. Bound by the output it writes. us for the 8-row form, before (whole tile's sums; stores of 32
// bytes per pixel) and now: 3 x 3 stride 2 in bf16, 32 channels, 1080 x 640 outputs 19.0 -> 15.0, 64 channels, stride 1,
// 1150 x 224 16.3 -> 12.9, fp32 3 x 640 x 640 x 64 121 -> 105. 7 x 7 in fp32 is bound by its matrix instructions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>

#include "act.hpp"
#include "conv_common.hpp"
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
  const float* bias;  // or nullptr
  int x_row0, x_rows, W;
  int y_row0, y_rows, W_out, C_out;
  int ph, pw, act, out_lo, R, N;
  int tiles_x, tiles_y;
  FastDiv by_x, by_y;
};

template <typename T, int KH> struct StemShape {
  static constexpr int KJ = 3 * KH;                          // elements of a filter row (three channels)
  static constexpr int KE = 16 / (int)sizeof(T);             // elements per group
  static constexpr int G = (KJ + KE - 1) / KE;               // groups per filter row
  static constexpr int STEPS = (KH * G + 1) / 2;
};

template <typename T, int KH, int S, int NT, int TH>
__device__ __forceinline__ void stem_body(const StemMfmaParams& p, const int bx) {
  using Sh = StemShape<T, KH>;
  constexpr int KE = Sh::KE, G = Sh::G, STEPS = Sh::STEPS, KJ = Sh::KJ;
  constexpr int EPD = 4 / (int)sizeof(T);                    // elements per 4-byte word
  constexpr int ROWS = (TH - 1) * S + KH;                    // image rows under the tile
  // words of a staged row: the last window's groups end inside it
  constexpr int WORDS = (((kTileCols - 1) * S * 3 + G * KE) + EPD - 1) / EPD + 1;
  constexpr int PITCH = WORDS | 1;                           // (odd: rows start on different banks)
  constexpr int COPIES = sizeof(T) == 2 && S == 1 ? 2 : 1;   // the second starts one element further on
  constexpr int RPW = (ROWS + 3) / 4, CPL = (WORDS + 63) / 64;
  constexpr int FW = TH / 2;                                 // 32-pixel fragments per wavefront
  __shared__ unsigned patch[COPIES][ROWS * PITCH];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, px = lane & 31;
  const int q = fastdiv(bx, p.by_x), tx = bx - q * p.tiles_x;
  const int n = fastdiv(q, p.by_y), ty = q - n * p.tiles_y;
  const int r0 = ty * TH, c0 = tx * kTileCols;

  // ---- stage: all loads first
  {
    const int ih0 = (p.out_lo + r0) * S - p.ph;
    const int e0 = (c0 * S - p.pw) * 3, row_elems = p.W * 3;
    unsigned v[COPIES][RPW][CPL];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const int r = wave + 4 * i, ih = ih0 + r;
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
          if (wave + 4 * i < ROWS && lane + 64 * j < WORDS) patch[c][(wave + 4 * i) * PITCH + lane + 64 * j] = v[c][i][j];
  }
  u32x4 w[STEPS][NT];
#pragma unroll
  for (int k = 0; k < NT; ++k)
#pragma unroll
    for (int t = 0; t < STEPS; ++t) w[t][k] = ((const u32x4*)p.w)[((size_t)(blockIdx.y * NT + k) * STEPS + t) * 64 + lane];
  __syncthreads();

  // ---- multiply. Group g: filter row g / G, elements (g % G) KE ..; step t is groups 2 t (lower half
  // of the wavefront) and 2 t + 1.
  // words of the last group of a filter row that hold elements of it
  auto last_mask = [](int j) constexpr {
    const int left = KJ - (G - 1) * KE - j * EPD;
    return left >= EPD ? 0xffffffffu : left <= 0 ? 0u : 0xffffu;
  };
  const unsigned upper = half ? 0xffffffffu : 0u;
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
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      constexpr int GROUPS = KH * G;
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

template <typename T, int KH, int S, int NT>
hipError_t launch_form(const OpLaunch* Ls, int n, bool large, hipStream_t s, KernelEvents* ev) {
  StemMfmaParams ps[kMaxBatch];
  unsigned gx[kMaxBatch];
  int m = 0;
  const int th = large ? 8 : 2;
  for (int b = 0; b < n; ++b) {
    const OpLaunch& L = Ls[b];
    StemMfmaParams p;
    p.x = L.x.ptr; p.y = L.y.ptr; p.y2 = L.y2; p.bias = L.bias;
    p.w = (const char*)L.wstem + stem_mfma_offset(L.x.c, L.y.c, L.kh, L.kw);
    p.x_row0 = L.x.row0; p.x_rows = L.x.rows; p.W = L.x.w;
    p.y_row0 = L.y.row0; p.y_rows = L.y.rows; p.W_out = L.y.w; p.C_out = L.y.c;
    p.ph = L.ph; p.pw = L.pw; p.act = L.act; p.out_lo = L.out_lo; p.R = L.out_hi - L.out_lo; p.N = L.x.n;
    if (p.R <= 0 || p.N <= 0) continue;
    p.tiles_x = (p.W_out + kTileCols - 1) / kTileCols;
    p.tiles_y = (p.R + th - 1) / th;
    p.by_x = make_fastdiv(p.tiles_x); p.by_y = make_fastdiv(p.tiles_y);
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

}  // namespace

bool stem_mfma_shape(int c_in, int c_out, int kh, int kw) { return c_in == 3 && c_out % 32 == 0 && kh == kw && (kh == 3 || kh == 7); }

size_t stem_mfma_offset(int c_in, int c_out, int kh, int kw) { return 2 * (size_t)c_out * c_in * kh * kw * sizeof(float); }

size_t stem_mfma_bytes(int c_out, int kh, int dtype) {
  const int steps = dtype == LOP_BF16 ? (kh == 3 ? StemShape<__bf16, 3>::STEPS : StemShape<__bf16, 7>::STEPS)
                                      : (kh == 3 ? StemShape<float, 3>::STEPS : StemShape<float, 7>::STEPS);
  return (size_t)(c_out / 32) * steps * 64 * 16;
}

// src: the packed rows [c_out][row_pitch], k = (a * kw + b) * 3 + ci, in the storage type
void stem_mfma_pack(const unsigned char* src, int row_pitch, int c_out, int kh, int dtype, unsigned char* dst) {
  if (dtype == LOP_BF16) kh == 3 ? pack<__bf16, 3>(src, row_pitch, c_out, dst) : pack<__bf16, 7>(src, row_pitch, c_out, dst);
  else kh == 3 ? pack<float, 3>(src, row_pitch, c_out, dst) : pack<float, 7>(src, row_pitch, c_out, dst);
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

}  // namespace lop
