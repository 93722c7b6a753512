// Bandwidth-bound local operators on a row interval: depthwise convolution, max pooling
// and the stand-alone element-wise operator (Intra-DP Sec. IV-A: block-wise and
// element-wise local operators). NHWC: a thread owns one 16-byte channel vector of one
// output pixel, consecutive threads own consecutive channel vectors, so every load and
// store of a wavefront is one contiguous run of channels. fp32 math, one rounding.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "act.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

struct RowParams {
  const void* x;
  void* y;
  void* y2;  // second destination with y's layout, or nullptr
  const void* res;
  const float* w;  // depthwise: [kh*kw][C] fp32
  const float* bias;
  int x_row0, x_rows, W, C;
  int y_row0, y_rows, W_out;
  int r_row0, r_rows;
  int kh, kw, sh, sw, ph, pw, dh, dw;
  int act, out_lo, R, N;
  long total;  // N * R * W_out * (C / VEC)
};

template <typename T, int VEC> struct Vec;  // VEC elements of T <-> fp32 registers

template <> struct Vec<float, 4> {
  static __device__ __forceinline__ void load(const float* p, float* v) {
    const float4 t = *(const float4*)p; v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
  static __device__ __forceinline__ void store(float* p, const float* v) {
    *(float4*)p = make_float4(v[0], v[1], v[2], v[3]);
  }
};
template <> struct Vec<float, 1> {
  static __device__ __forceinline__ void load(const float* p, float* v) { v[0] = *p; }
  static __device__ __forceinline__ void store(float* p, const float* v) { *p = v[0]; }
};
template <> struct Vec<__bf16, 8> {
  static __device__ __forceinline__ void load(const __bf16* p, float* v) {
    const uint4 t = *(const uint4*)p;
    const unsigned u[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(u[i] << 16);
      v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ void store(__bf16* p, const float* v) {
    alignas(16) __bf16 o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (__bf16)v[i];
    *(uint4*)p = *(const uint4*)o;
  }
};
template <> struct Vec<__bf16, 4> {
  static __device__ __forceinline__ void load(const __bf16* p, float* v) {
    const uint2 t = *(const uint2*)p;
    v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
    v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
  }
  static __device__ __forceinline__ void store(__bf16* p, const float* v) {
    alignas(8) __bf16 o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = (__bf16)v[i];
    *(uint2*)p = *(const uint2*)o;
  }
};
template <> struct Vec<__bf16, 1> {
  static __device__ __forceinline__ void load(const __bf16* p, float* v) { v[0] = (float)*p; }
  static __device__ __forceinline__ void store(__bf16* p, const float* v) { *p = (__bf16)v[0]; }
};

template <int VEC>
__device__ __forceinline__ void load_f32(const float* p, float* v) {
  if constexpr (VEC >= 4) {
#pragma unroll
    for (int i = 0; i < VEC; i += 4) {
      const float4 t = *(const float4*)(p + i);
      v[i] = t.x; v[i + 1] = t.y; v[i + 2] = t.z; v[i + 3] = t.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i) v[i] = p[i];
  }
}

// OP: 0 depthwise conv, 1 max pool, 2 element-wise
template <typename T, int VEC, int OP>
__device__ __forceinline__ void rowwise_kernel_body(const RowParams& p, const int bx) {
  const long gid = (long)bx * 256 + threadIdx.x;
  if (gid >= p.total) return;
  const int cv = p.C / VEC;
  const int c = (int)(gid % cv) * VEC;
  long t = gid / cv;
  const int ow = (int)(t % p.W_out);
  t /= p.W_out;
  const int r = (int)(t % p.R), n = (int)(t / p.R);
  const int oh = p.out_lo + r;
  const T* __restrict__ xg = (const T*)p.x;
  float acc[VEC];
  if (OP == 2) {
    Vec<T, VEC>::load(xg + ((size_t)(n * p.x_rows + oh - p.x_row0) * p.W + ow) * p.C + c, acc);
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = OP == 1 ? -INFINITY : 0.f;
    const int ih0 = oh * p.sh - p.ph, iw0 = ow * p.sw - p.pw;
    for (int a = 0; a < p.kh; ++a) {
      const int ih = ih0 + a * p.dh;
      if (ih < p.x_row0 || ih >= p.x_row0 + p.x_rows) continue;
      for (int b = 0; b < p.kw; ++b) {
        const int iw = iw0 + b * p.dw;
        if (iw < 0 || iw >= p.W) continue;
        float v[VEC];
        Vec<T, VEC>::load(xg + ((size_t)(n * p.x_rows + ih - p.x_row0) * p.W + iw) * p.C + c, v);
        if (OP == 1) {
#pragma unroll
          for (int i = 0; i < VEC; ++i) acc[i] = fmaxf(acc[i], v[i]);
        } else {
          float wv[VEC];
          load_f32<VEC>(p.w + (size_t)(a * p.kw + b) * p.C + c, wv);
#pragma unroll
          for (int i = 0; i < VEC; ++i) acc[i] = fmaf(v[i], wv[i], acc[i]);
        }
      }
    }
  }
  if (OP != 1) {
    if (p.bias) {
      float bv[VEC];
      load_f32<VEC>(p.bias + c, bv);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] += bv[i];
    }
    if (p.res) {
      float rv[VEC];
      Vec<T, VEC>::load((const T*)p.res +
                            ((size_t)(n * p.r_rows + oh - p.r_row0) * p.W_out + ow) * p.C + c, rv);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] += rv[i];
    }
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = clamp_act(acc[i], make_clamp(p.act));
  }
  const size_t yo = ((size_t)(n * p.y_rows + oh - p.y_row0) * p.W_out + ow) * p.C + c;
  Vec<T, VEC>::store((T*)p.y + yo, acc);
  if (p.y2) Vec<T, VEC>::store((T*)p.y2 + yo, acc);
}

template <typename T, int VEC, int OP>
__global__ __launch_bounds__(256) void rowwise_kernel(const RowParams p) {
  rowwise_kernel_body<T, VEC, OP>(p, blockIdx.x);
}
// The same for several bands of one layer in one grid (band b owns blocks first[b] .. first[b + 1]).
template <typename T, int VEC, int OP>
__global__ __launch_bounds__(256) void rowwise_kernel_bands(const Batch<RowParams> t) {
  const int b = batch_find(t, blockIdx.x);
  rowwise_kernel_body<T, VEC, OP>(t.p[b], blockIdx.x - t.first[b]);
}


// Depthwise 3x3 (dilation 1, pad 1, stride S in both directions), register blocked: a
// thread owns VEC channels of COLS neighbouring output columns (see dw_cols) and dw_rows_per_thread(S) consecutive output
// rows; it loads the (rows-1)*S + 3 input rows it needs, (COLS-1)*S + 3 vectors each, and the 9 x VEC
// weights once, so an output costs 3.75 vector loads with stride 1 and 6.75 with stride 2 (one column), 2.5 and 5.6 (two), instead
// of 9 loads plus 9 weight loads. Threads of a workgroup are (channel vector, column) with the channel
// vector fastest: loads and stores of a wavefront stay contiguous and the left/right
// neighbours' columns come out of the same CU's L1. No residual (rowwise_kernel has it).
// Output rows per thread: the (rows - 1) * S + 3 input rows are read once per thread, so the
// rows shared with the chunk above and below are fetched twice: 6 for 4 with stride 1 (1.5 x),
// 10 for 8 (1.25 x); with stride 2, 9 for 4 is 1.125 x already.
constexpr int dw_rows_per_thread(int stride) { return stride == 1 ? 8 : 4; }
struct Dw3Params {
  RowParams r;
  int cols_per_block;  // output columns per workgroup
  int col_blocks;      // workgroups per row chunk
  int chunks;          // row chunks (dw_rows_per_thread output rows each) per image
};
static_assert(sizeof(Batch<Dw3Params>) <= 4096, "the parameters of all bands of a launch travel as kernel arguments");

// Raw 8- or 16-byte vector of the storage type and its expansion to fp32 values.
template <int BYTES> struct RawVec;
template <> struct RawVec<16> { typedef unsigned type __attribute__((ext_vector_type(4))); };
template <> struct RawVec<8> { typedef unsigned type __attribute__((ext_vector_type(2))); };
typedef RawVec<16>::type raw16;
typedef RawVec<8>::type raw8;
__device__ __forceinline__ raw16 raw_load(__amdgpu_buffer_rsrc_t buf, unsigned at, raw16) { return __builtin_amdgcn_raw_buffer_load_b128(buf, (int)at, 0, 0); }
__device__ __forceinline__ raw8 raw_load(__amdgpu_buffer_rsrc_t buf, unsigned at, raw8) { return __builtin_amdgcn_raw_buffer_load_b64(buf, (int)at, 0, 0); }
__device__ __forceinline__ void raw_store(const raw16& v, __amdgpu_buffer_rsrc_t buf, unsigned at) { __builtin_amdgcn_raw_buffer_store_b128(v, buf, (int)at, 0, 0); }
__device__ __forceinline__ void raw_store(const raw8& v, __amdgpu_buffer_rsrc_t buf, unsigned at) { __builtin_amdgcn_raw_buffer_store_b64(v, buf, (int)at, 0, 0); }

__device__ __forceinline__ void unpack_bf16(const raw8& t, float* v) {
  v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
}
__device__ __forceinline__ void unpack_f32(const raw16& t, float* v) {
  v[0] = __uint_as_float(t.x); v[1] = __uint_as_float(t.y);
  v[2] = __uint_as_float(t.z); v[3] = __uint_as_float(t.w);
}
template <typename T, typename R>
__device__ __forceinline__ void unpack(const R& t, float* v) {
  if constexpr (sizeof(T) == 2) unpack_bf16(t, v);
  else unpack_f32(t, v);
}

// COLS: columns of outputs per thread, which share the input columns between them.
template <typename T, int VEC, int S, int COLS>
__device__ __forceinline__ void dwconv3x3_body(const Dw3Params& q, const int bx) {
  static_assert(VEC * sizeof(T) == 16 || VEC * sizeof(T) == 8, "8- or 16-byte vectors");
  typedef typename RawVec<VEC * sizeof(T)>::type Raw;
  constexpr int RPT = dw_rows_per_thread(S);  // output rows per thread
  constexpr int NR = (RPT - 1) * S + 3;    // input rows they read
  constexpr int NC = (COLS - 1) * S + 3;   // input columns
  const RowParams& p = q.r;
  const int cv = p.C / VEC;
  const int cg = threadIdx.x % cv, col = threadIdx.x / cv * COLS;
  const int row = bx / q.col_blocks;
  const int ow_first = (bx - row * q.col_blocks) * q.cols_per_block, ow = ow_first + col;   // of the workgroup, of the thread
  if (col >= q.cols_per_block || ow >= p.W_out) return;
  const int n = row / q.chunks, chunk = row - n * q.chunks;
  const int c = cg * VEC;
  const int oh0 = p.out_lo + chunk * RPT;
  const int oh1 = min(oh0 + RPT, p.out_lo + p.R);
  const Clamp clamp = make_clamp(p.act);

  // Every load first (input rows, weights, bias), all stores after: loads and stores share
  // one in-order counter, so a load waited for after a store would wait for the store too.
  // A row is a buffer of its own, from the workgroup's first column to the row's end: columns outside the image and rows outside
  // the slab (buffers of no bytes) read as zeros.
  const int pixel = p.C * (int)sizeof(T), iw_first = max(ow_first * S - 1, 0);
  const size_t x_pitch = (size_t)p.W * pixel, y_pitch = (size_t)p.W_out * pixel;
  auto up_to_end = [&](int columns) { return (int)min((size_t)columns * pixel, (size_t)0x7fffffff); };
  const int x_bytes = up_to_end(p.W - iw_first), y_bytes = up_to_end(p.W_out - ow_first);
  Raw in[NR][NC];
  const int ih0 = oh0 * S - 1;
  const int rows_needed = (oh1 - oh0 - 1) * S + 3;
  const unsigned x_at = (unsigned)((ow * S - 1 - iw_first) * pixel + c * (int)sizeof(T));
#pragma unroll
  for (int a = 0; a < NR; ++a) {
    const int ih = ih0 + a;
    const bool row_ok = a < rows_needed && ih >= p.x_row0 && ih < p.x_row0 + p.x_rows;
    const __amdgpu_buffer_rsrc_t buf = __builtin_amdgcn_make_buffer_rsrc(
        (char*)const_cast<void*>(p.x) + (row_ok ? (size_t)(n * p.x_rows + ih - p.x_row0) * x_pitch + (size_t)iw_first * pixel : (size_t)0), 0,
        row_ok ? x_bytes : 0, 0x00020000);
#pragma unroll
    for (int b = 0; b < NC; ++b) in[a][b] = raw_load(buf, x_at + b * pixel, Raw{});
  }
  float w[9][VEC];
#pragma unroll
  for (int t = 0; t < 9; ++t) load_f32<VEC>(p.w + (size_t)t * p.C + c, w[t]);
  float bias[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) bias[i] = 0.f;
  if (p.bias) load_f32<VEC>(p.bias + c, bias);

  float x[3][NC][VEC];   // the rows under one output row: each is unpacked once
  const unsigned y_at = (unsigned)(col * pixel + c * (int)sizeof(T));
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    if (oh0 + r >= oh1) break;
#pragma unroll
    for (int a = r == 0 ? 0 : 3 - S; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < NC; ++b) unpack<T>(in[r * S + a][b], x[(r * S + a) % 3][b]);
    const size_t y_row = (size_t)(n * p.y_rows + oh0 + r - p.y_row0) * y_pitch + (size_t)ow_first * pixel;
    const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc((char*)p.y + y_row, 0, y_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t to2 = __builtin_amdgcn_make_buffer_rsrc((char*)p.y2 + (p.y2 ? y_row : 0), 0, p.y2 ? y_bytes : 0, 0x00020000);
#pragma unroll
    for (int k = 0; k < COLS; ++k) {
      float acc[VEC];
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] = bias[i];
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
          for (int i = 0; i < VEC; ++i) acc[i] = fmaf(x[(r * S + a) % 3][k * S + b][i], w[a * 3 + b][i], acc[i]);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] = clamp_act(acc[i], clamp);
      alignas(16) T o[VEC];
      Vec<T, VEC>::store(o, acc);
      raw_store(*(const Raw*)o, to, y_at + k * pixel);   // (past the row's end: nowhere)
      if (p.y2) raw_store(*(const Raw*)o, to2, y_at + k * pixel);
    }
  }
}

template <typename T> constexpr int kDwCols = sizeof(T) == 2 ? 2 : 1;
template <typename T, int VEC, int S>
__global__ __launch_bounds__(256) void dwconv3x3_kernel(const Dw3Params q) {
  dwconv3x3_body<T, VEC, S, kDwCols<T>>(q, blockIdx.x);
}
// The same for several bands of one layer in one grid (band b owns blocks first[b] .. first[b + 1]).
template <typename T, int VEC, int S>
__global__ __launch_bounds__(256) void dwconv3x3_kernel_bands(const Batch<Dw3Params> t) {
  const int b = batch_find(t, blockIdx.x);
  dwconv3x3_body<T, VEC, S, kDwCols<T>>(t.p[b], blockIdx.x - t.first[b]);
}
// bf16 with one column a thread, for launches of few workgroups (see dw_cols).
template <typename T, int VEC, int S>
__global__ __launch_bounds__(256) void dwconv3x3_column_kernel(const Dw3Params q) {
  dwconv3x3_body<T, VEC, S, 1>(q, blockIdx.x);
}
template <typename T, int VEC, int S>
__global__ __launch_bounds__(256) void dwconv3x3_column_kernel_bands(const Batch<Dw3Params> t) {
  const int b = batch_find(t, blockIdx.x);
  dwconv3x3_body<T, VEC, S, 1>(t.p[b], blockIdx.x - t.first[b]);
}

// The sliding-window kernel covers the common depthwise case; everything else runs on
// rowwise_kernel.
inline bool dw3_applies(const RowParams& p, int op, int vec) {
  return op == LOP_DWCONV2D && p.kh == 3 && p.kw == 3 && p.dh == 1 && p.dw == 1 && p.ph == 1 &&
         p.pw == 1 && p.sh == p.sw && (p.sh == 1 || p.sh == 2) && vec > 1 && p.C / vec <= 256 &&
         p.res == nullptr;
}

constexpr int kDwVec = 4;   // channels per thread
inline int dw_block_cols(int c, int cols) { return std::max(1, 256 / (c / kDwVec)) * cols; }

// Columns of outputs per thread of a launch: two (bf16; fp32 has no registers for them) where that leaves a workgroup per
// compute unit. Two take 2.5 vector loads an output where one takes 3.75 (stride 2: 5.6 and 6.75) and half the vector
// instructions, which were busy for three quarters of the time: 192 channels on 8 x 42 x 320 pixels 26.9 -> 22.2 us, stride 2 on
// 8 x 82 x 640 42.5 -> 39.8. With few workgroups a thread's chain of loads is what counts: 2 x 20 x 84 pixels 4.5 us with
// one column, 5.8 with two; 42 x 160 (96 workgroups of two) 4.7 and 5.9. Between them one is ahead alone up to one and a half
// to a compute unit (us a launch, one and two columns: 144 x 144 pixels, 270 workgroups, 7.7 and 8.3; 160 x 160, 320, 8.2 and 8.7; stride 2 on 224 x
// 224, 336, 6.8 and 7.3; 8 x 21 x 160, 384, 8.4 and 8.7; but 176 x 176, 396, 9.5 and 9.0; stride 2 on 256 x 256, 416, 7.9 and 7.5), two
// with launches beside it (chains of one 640 x 640 image in four bands 262.9 and 258.2 us, of eight in eight bands 1 959 and 1 942).
// So where the line lies depends on whose stream the chain runs on.
constexpr long kDwTwoColumns = 256, kDwTwoColumnsAlone = 384;
int dw_cols(const RowParams* ps, int n, int dtype, bool alone) {
  long blocks = 0;
  for (int b = 0; b < n; ++b) {
    const RowParams& p = ps[b];
    if (p.R <= 0 || p.N <= 0) continue;
    const int rpt = dw_rows_per_thread(p.sh), cols = dw_block_cols(p.C, 2);
    blocks += (long)((p.W_out + cols - 1) / cols) * ((p.R + rpt - 1) / rpt) * p.N;
  }
  return dtype == LOP_BF16 && blocks > (alone ? kDwTwoColumnsAlone : kDwTwoColumns) ? 2 : 1;
}

// The bands in one launch, unless they have more workgroups than a launch takes (2^32 threads, exclusive): then in as few as
// hold them, a band of too many itself cut into groups of images or of rows of an image.
constexpr long kDwBlocks = 0xffffffffL / 256;
template <typename T, int VEC, int COLS>
hipError_t launch_dw3(const RowParams* ps, int n, hipStream_t s, KernelEvents* ev) {
  Dw3Params qs[kMaxBatch];
  unsigned gx[kMaxBatch];
  int m = 0;
  long total = 0;
  auto launch = [&]() -> hipError_t {
    const int k = m;
    m = 0; total = 0;
    if (k == 0) return hipSuccess;
    const dim3 block(256);
    if constexpr (COLS != kDwCols<T>) {
      return ps[0].sh == 1 ? launch_group(dwconv3x3_column_kernel<T, VEC, 1>, dwconv3x3_column_kernel_bands<T, VEC, 1>, qs, k, gx, 1, 1, block, s, ev)
                           : launch_group(dwconv3x3_column_kernel<T, VEC, 2>, dwconv3x3_column_kernel_bands<T, VEC, 2>, qs, k, gx, 1, 1, block, s, ev);
    } else {
      return ps[0].sh == 1 ? launch_group(dwconv3x3_kernel<T, VEC, 1>, dwconv3x3_kernel_bands<T, VEC, 1>, qs, k, gx, 1, 1, block, s, ev)
                           : launch_group(dwconv3x3_kernel<T, VEC, 2>, dwconv3x3_kernel_bands<T, VEC, 2>, qs, k, gx, 1, 1, block, s, ev);
    }
  };
  for (int b = 0; b < n; ++b) {
    const RowParams& p = ps[b];
    if (p.R <= 0 || p.N <= 0) continue;
    const int rpt = dw_rows_per_thread(p.sh), cols = dw_block_cols(p.C, COLS), col_blocks = (p.W_out + cols - 1) / cols;
    // (not even one chunk of rows with a column a thread: an error whichever form is taken)
    if ((p.W_out + dw_block_cols(p.C, 1) - 1) / dw_block_cols(p.C, 1) > kDwBlocks) return hipErrorInvalidValue;
    const int rows = (int)std::min((long)p.R, kDwBlocks / col_blocks * rpt);
    const int images = (int)std::min((long)p.N, kDwBlocks / ((long)col_blocks * ((rows + rpt - 1) / rpt)));
    const size_t x_img = (size_t)p.x_rows * p.W * p.C * sizeof(T), y_img = (size_t)p.y_rows * p.W_out * p.C * sizeof(T);
    for (int i = 0; i < p.N; i += images)
      for (int r = 0; r < p.R; r += rows) {
        Dw3Params q;
        q.r = p;
        q.r.x = (const char*)p.x + i * x_img;
        q.r.y = (char*)p.y + i * y_img;
        q.r.y2 = p.y2 ? (char*)p.y2 + i * y_img : nullptr;
        q.r.N = std::min(images, p.N - i);
        q.r.out_lo = p.out_lo + r;
        q.r.R = std::min(rows, p.R - r);
        q.cols_per_block = cols;
        q.col_blocks = col_blocks;
        q.chunks = (q.r.R + rpt - 1) / rpt;
        const long blocks = (long)col_blocks * q.chunks * q.r.N;
        if (m == kMaxBatch || total + blocks > kDwBlocks) {
          const hipError_t e = launch();
          if (e != hipSuccess) return e;
        }
        qs[m] = q;
        gx[m++] = (unsigned)blocks;
        total += blocks;
      }
  }
  return launch();
}

// Channel vector per thread of the sliding-window kernel (0: it does not apply).
inline int dw3_vec(const RowParams& p, int op) {
  if (p.C % kDwVec != 0) return 0;
  return dw3_applies(p, op, kDwVec) ? kDwVec : 0;
}

template <typename T, int VEC>
hipError_t launch_rowwise(RowParams* ps, int n, int op, hipStream_t s, KernelEvents* ev) {
  unsigned gx[kMaxBatch];
  int m = 0;
  for (int b = 0; b < n; ++b) {
    ps[b].total = (long)ps[b].N * ps[b].R * ps[b].W_out * (ps[b].C / VEC);
    if (ps[b].total <= 0) continue;
    ps[m] = ps[b];
    gx[m++] = (unsigned)((ps[b].total + 255) / 256);
  }
  if (m == 0) return hipSuccess;
  if (op == LOP_DWCONV2D)
    return launch_group(rowwise_kernel<T, VEC, 0>, rowwise_kernel_bands<T, VEC, 0>, ps, m, gx, 1, 1, dim3(256), s, ev);
  if (op == LOP_MAXPOOL2D)
    return launch_group(rowwise_kernel<T, VEC, 1>, rowwise_kernel_bands<T, VEC, 1>, ps, m, gx, 1, 1, dim3(256), s, ev);
  return launch_group(rowwise_kernel<T, VEC, 2>, rowwise_kernel_bands<T, VEC, 2>, ps, m, gx, 1, 1, dim3(256), s, ev);
}

RowParams make_row_params(const OpLaunch& L) {
  RowParams p;
  p.x = L.x.ptr; p.y = L.y.ptr; p.y2 = L.y2; p.res = L.res.ptr; p.w = (const float*)L.w; p.bias = L.bias;
  p.x_row0 = L.x.row0; p.x_rows = L.x.rows; p.W = L.x.w; p.C = L.x.c;
  p.y_row0 = L.y.row0; p.y_rows = L.y.rows; p.W_out = L.y.w;
  p.r_row0 = L.res.row0; p.r_rows = L.res.rows;
  p.kh = L.kh; p.kw = L.kw; p.sh = L.sh; p.sw = L.sw; p.ph = L.ph; p.pw = L.pw;
  p.dh = L.dh; p.dw = L.dw;
  p.act = L.act; p.out_lo = L.out_lo; p.R = L.out_hi - L.out_lo; p.N = L.x.n;
  p.total = 0;
  return p;
}

}  // namespace

// The register-blocked depthwise kernel.
bool dw3_takes(const OpLaunch& L) { return dw3_vec(make_row_params(L), L.op) != 0; }

hipError_t launch_rowwise_bands(const OpLaunch* Ls, int n, hipStream_t stream, KernelEvents* ev) {
  if (n < 1 || n > kMaxBatch) return hipErrorInvalidValue;
  RowParams ps[kMaxBatch];
  for (int b = 0; b < n; ++b) ps[b] = make_row_params(Ls[b]);
  const OpLaunch& L = Ls[0];
  RowParams& p = ps[0];
  if (dw3_vec(p, L.op))
    return L.dtype != LOP_BF16 ? launch_dw3<float, kDwVec, 1>(ps, n, stream, ev)
           : dw_cols(ps, n, L.dtype, L.alone) == 2 ? launch_dw3<__bf16, kDwVec, 2>(ps, n, stream, ev)
                                          : launch_dw3<__bf16, kDwVec, 1>(ps, n, stream, ev);
  if (L.dtype == LOP_BF16)
    return p.C % 8 == 0 ? launch_rowwise<__bf16, 8>(ps, n, L.op, stream, ev)
                        : launch_rowwise<__bf16, 1>(ps, n, L.op, stream, ev);
  return p.C % 4 == 0 ? launch_rowwise<float, 4>(ps, n, L.op, stream, ev)
                      : launch_rowwise<float, 1>(ps, n, L.op, stream, ev);
}

hipError_t launch_rowwise_op(const OpLaunch& L, hipStream_t stream, KernelEvents* ev) {
  return launch_rowwise_bands(&L, 1, stream, ev);
}

namespace {
// Copies `n` segments of `len` bytes (segment i at offset i*pitch in both buffers), 16 bytes
// per thread and step. Used to push finished rows into mapped pinned host memory: the stores
// travel over PCIe while other streams compute. Non-temporal in both directions: nobody reads
// either side again here, and rows on their way to the host that go through the caches push out
// what the kernels beside the copy use (the 720p chain in reuse mode 77 -> 72 us).
constexpr int kCopyThreads = 512;
__global__ __launch_bounds__(kCopyThreads) void copy_rows_kernel(char* __restrict__ dst,
                                                        const char* __restrict__ src,
                                                        size_t pitch, size_t len, int n) {
  typedef unsigned vec_t __attribute__((ext_vector_type(4)));
  const size_t vec = len / 16;
  const size_t stride = (size_t)gridDim.x * kCopyThreads;
  for (int i = 0; i < n; ++i) {
    const vec_t* s = (const vec_t*)(src + i * pitch);
    vec_t* d = (vec_t*)(dst + i * pitch);
    for (size_t j = (size_t)blockIdx.x * kCopyThreads + threadIdx.x; j < vec; j += stride)
      __builtin_nontemporal_store(__builtin_nontemporal_load(s + j), d + j);
    // tail bytes (len is a multiple of the element size, not necessarily of 16)
    for (size_t j = vec * 16 + (size_t)blockIdx.x * kCopyThreads + threadIdx.x; j < len; j += stride)
      dst[i * pitch + j] = src[i * pitch + j];
  }
}
// Fills `bytes` (a multiple of 16) with one 32-bit pattern: the debug poisoning of scratch
// memory (a kernel, not a memset, so that it may be captured into a graph).
__global__ __launch_bounds__(256) void fill_words_kernel(uint4* __restrict__ dst, size_t vecs, unsigned word) {
  const size_t stride = (size_t)gridDim.x * 256;
  const uint4 v = make_uint4(word, word, word, word);
  for (size_t j = (size_t)blockIdx.x * 256 + threadIdx.x; j < vecs; j += stride) dst[j] = v;
}
}  // namespace

hipError_t launch_fill_words(void* dst, size_t bytes, unsigned word, hipStream_t stream) {
  const size_t vecs = bytes / 16;
  if (!dst || vecs == 0) return hipSuccess;
  const unsigned grid = (unsigned)std::min<size_t>((vecs + 255) / 256, 2048);
  hipLaunchKernelGGL(fill_words_kernel, dim3(grid), dim3(256), 0, stream, (uint4*)dst, vecs, word);
  return hipGetLastError();
}

hipError_t launch_copy_rows(void* dst, const void* src, size_t pitch, size_t len, int n,
                            hipStream_t stream, int workgroups) {
  if (len == 0 || n <= 0) return hipSuccess;
  const size_t vec = (len + 15) / 16;
  // Few workgroups on purpose (see the caller's number)
  const unsigned grid = (unsigned)std::min<size_t>((vec + kCopyThreads - 1) / kCopyThreads, (size_t)std::max(1, workgroups));
  hipLaunchKernelGGL(copy_rows_kernel, dim3(grid), dim3(kCopyThreads), 0, stream, (char*)dst,
                     (const char*)src, pitch, len, n);
  return hipGetLastError();
}

int rowwise_describe(const OpLaunch& L, char* name, size_t size) {
  const bool bf = L.dtype == LOP_BF16;
  const int vec = bf ? (L.x.c % 8 == 0 ? 8 : 1) : (L.x.c % 4 == 0 ? 4 : 1);
  const int o = L.op == LOP_DWCONV2D ? 0 : (L.op == LOP_MAXPOOL2D ? 1 : 2);
  RowParams p;
  p.kh = L.kh; p.kw = L.kw; p.sh = L.sh; p.sw = L.sw; p.ph = L.ph; p.pw = L.pw;
  p.dh = L.dh; p.dw = L.dw; p.C = L.x.c; p.res = L.res.ptr;
  p.W = L.x.w; p.W_out = L.y.w; p.R = L.out_hi - L.out_lo; p.N = L.x.n;
  if (name && size) {
    if (const int v = dw3_vec(p, L.op))
      snprintf(name, size, "dwconv3x3_%skernel<%s, %d, %d>", bf && dw_cols(&p, 1, L.dtype, L.alone) == 1 ? "column_" : "", bf ? "__bf16" : "float", v, L.sh);
    else
      snprintf(name, size, "rowwise_kernel<%s, %d, %d>", bf ? "__bf16" : "float", vec, o);
  }
  return 1;
}

}  // namespace lop
