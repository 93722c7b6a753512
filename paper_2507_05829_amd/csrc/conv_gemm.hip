// Dense 1 x 1 convolution (any stride; the row-wise operator of Eq. 1) as a tiled matrix product
// with both operands travelling global -> LDS without passing through registers.
//
// A workgroup of WM x WN wavefronts owns BM pixels x BN channels; NST stages of 128 bytes of the
// reduction per row sit in LDS, fetched by loads that cover 8 rows x 128 bytes each. What the loop is
// built around: a compute unit's matrix cores need both wavefronts of a SIMD to have an MFMA ready
// all the time, so
//  - the fragments of the next 32 bytes of the reduction are read from LDS while the current ones are
//    multiplied, across stages, too: the barrier that opens the next stage stands in front of the last
//    multiply of the current one, and behind it the next stage's first fragments are already on their
//    way;
//  - one barrier per stage. Behind it no wavefront reads the current stage any more (its last
//    fragments are in registers), so its memory is refilled at once with the stage NST further on;
//  - the reads are instructions of our own (reads the compiler can see make it wait for every load
//    to LDS that is in flight), the waits are placed by hand.
// A row's 16-byte chunks are stored at chunk ^ (row / 2 mod 8): the 16 lanes that read one chunk of 16
// neighbouring rows at a time touch every LDS bank once. A row past the launch's pixels or a chunk past
// the end of the reduction is a load past the end of the buffer resource and arrives as zeros.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>

#include "act.hpp"
#include "conv_common.hpp"
#include "conv_split.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

struct GemmParams {
  const void* x;
  void* y;
  void* y2;        // second destination with y's layout, or nullptr
  const void* res;
  const void* w;   // [c_out_pad][k_pad]; where the products are made of parts: the operand-order packing
  const void* w3;  // the same weights as three bf16 parts in operand order (fp32 layers)
  const float* bias;
  int x_row0, x_rows, W, K;          // K: channels in
  int y_row0, y_rows, W_out, C_out;
  int r_row0, r_rows;
  int sh, sw, ph, pw, act, k_pad;
  int out_lo, R, N, M;               // M = N * R * W_out
  int mx, ny;                        // tiles of a launch that walks over them, else 0
  FastDiv by_w, by_r, by_group;
};
static_assert(sizeof(Batch<GemmParams>) <= 4096, "the parameters of all bands of a launch travel as kernel arguments");

constexpr unsigned kOutside = 0x80000000u;
constexpr int gemm_pitch(int tn) { return tn * 32 + 4; }   // fp32 elements of a row of a wavefront's staged output tile

// What follows the sums: one 32-pixel tile of the wavefront at a time through LDS, so that consecutive lanes
// own consecutive 16-byte pieces of a pixel's channels. (The caller's barrier lies between smem's last readers and this.)
template <typename T, int TM, int TN>
__device__ __forceinline__ void gemm_epilogue(const GemmParams& p, unsigned char* smem, const f32x16 (&acc)[TN][TM], int m0, int co0,
                                              int wave, int wm, int wn, int lane) {
  constexpr int CPW = gemm_pitch(TN);
  constexpr int VE = 16 / (int)sizeof(T);
  constexpr int CPR = TN * 32 / VE;          // pieces per pixel of the wavefront's tile
  float* const Cw = (float*)smem + wave * (32 * CPW);
  const Clamp cl = make_clamp(p.act);
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    constexpr int PIECES = 32 * CPR / 64;
    // the residual's pieces (and where they go) first: their latency passes under the exchange
    size_t ya[PIECES];
    u32x4 rr[PIECES];
    bool ok[PIECES];
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int slot = lane + i * 64, row = slot / CPR, c = (slot % CPR) * VE;
      const int m = m0 + (wm * TM + tm) * 32 + row, co = co0 + wn * TN * 32 + c;
      ok[i] = (m < p.M) & (co < p.C_out);
      const int mm = ok[i] ? m : 0;
      const int q = fastdiv(mm, p.by_w), ow = mm - q * p.W_out;
      const int n = fastdiv(q, p.by_r), oh = p.out_lo + q - n * p.R;
      ya[i] = ((size_t)(n * p.y_rows + oh - p.y_row0) * p.W_out + ow) * p.C_out + co;
      rr[i] = u32x4{0u, 0u, 0u, 0u};
      if (p.res && ok[i]) rr[i] = *(const u32x4*)((const T*)p.res + ((size_t)(n * p.r_rows + oh - p.r_row0) * p.W_out + ow) * p.C_out + co);
    }
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(f32x4*)(Cw + (lane & 31) * CPW + tn * 32 + g * 8 + (lane >> 5) * 4) =
            f32x4{acc[tn][tm][g * 4], acc[tn][tm][g * 4 + 1], acc[tn][tm][g * 4 + 2], acc[tn][tm][g * 4 + 3]};
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int slot = lane + i * 64, row = slot / CPR, c = (slot % CPR) * VE;
      if (!ok[i]) continue;
      alignas(16) T in[VE], o[VE];
      *(u32x4*)in = rr[i];
#pragma unroll
      for (int j = 0; j < VE; j += 4) {
        f32x4 v = *(const f32x4*)(Cw + row * CPW + c + j);
        if (p.bias) v += *(const f32x4*)(p.bias + co0 + wn * TN * 32 + c + j);
#pragma unroll
        for (int k = 0; k < 4; ++k) o[j + k] = from_f32<T>(clamp_act(v[k] + to_f32(in[j + k]), cl));
      }
      *(u32x4*)((T*)p.y + ya[i]) = *(const u32x4*)o;
      if (p.y2) *(u32x4*)((T*)p.y2 + ya[i]) = *(const u32x4*)o;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// The same from registers, without LDS, residual or second destination: a lane holds channels 8 g + 4 half + {0..3} of pixel lane mod 32 of a 32 x 32
// tile; exchanges between the lane halves and between rows of 16 lanes make each store write 64 consecutive bytes of
// 16 pixels. (As fast as the form above within 2 %; two stores of every lane per 32 x 32 tile where all of it lies inside.)
template <typename T, int TM, int TN>
__device__ __forceinline__ void gemm_store(const GemmParams& p, const f32x16 (&acc)[TN][TM], const f32x4 (&bias)[TN][4], int m_first,
                                           int co_first, int lane) {
  static_assert(sizeof(T) == 2, "bf16");
  const int half = lane >> 5;
  const int piece = half + ((lane >> 4) & 1) * 2;          // of the four of a store's 64 bytes
  const Clamp cl = make_clamp(p.act);
  auto pixel = [&](int m) __attribute__((always_inline)) {   // offset of a pixel's first channel
    const int mm = m < p.M ? m : 0;
    const int q = fastdiv(mm, p.by_w), ow = mm - q * p.W_out;
    const int n = fastdiv(q, p.by_r), oh = p.out_lo + q - n * p.R;
    return ((size_t)(n * p.y_rows + oh - p.y_row0) * p.W_out + ow) * p.C_out;
  };
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    const int m = m_first + tm * 32 + (lane & 15);
    const size_t at[2] = {pixel(m), pixel(m + 16)};
    const bool live[2] = {m < p.M, m + 16 < p.M};
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      const int co = co_first + tn * 32;
      u32x4 o[2];
#pragma unroll
      for (int g = 0; g < 4; g += 2) {
        alignas(16) __bf16 b[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          f32x4 v = f32x4{acc[tn][tm][(g + h) * 4], acc[tn][tm][(g + h) * 4 + 1], acc[tn][tm][(g + h) * 4 + 2], acc[tn][tm][(g + h) * 4 + 3]};
          v += bias[tn][g + h];
#pragma unroll
          for (int k = 0; k < 4; ++k) b[h * 4 + k] = from_f32<T>(clamp_act(v[k], cl));
        }
        const u32x4 w = *(const u32x4*)b;
        const auto s0 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
        o[g / 2] = u32x4{(unsigned)s0[0], (unsigned)s1[0], (unsigned)s0[1], (unsigned)s1[1]};
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const auto s = __builtin_amdgcn_permlane16_swap(o[0][j], o[1][j], false, false);
        o[0][j] = s[0];
        o[1][j] = s[1];
      }
      const int c = co + piece * 8;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (live[h] & (c < p.C_out)) *(u32x4*)((T*)p.y + at[h] + c) = o[h];
    }
  }
}

// LDS of a workgroup: the stages, later the staged output tiles.
template <int BM, int BN, int WM, int WN, int NST>
constexpr int gemm_smem() {
  constexpr int stages = NST * (BM + BN) * 128, out = WM * WN * 32 * gemm_pitch(BN / (32 * WN)) * 4;
  static_assert(stages <= 160 * 1024 && out <= 160 * 1024, "LDS");
  return stages > out ? stages : out;
}

// WALK: the workgroup takes tiles launch, launch + step, ... of mx * ny (else the first of them only). Its loop needs all the
// LDS a compute unit has, so that no other workgroup hides a tile's start and end: 3.8 us of the 35 that 16 stages take. The next
// tile's first stages are therefore on their way while this one's sums leave, from registers. (A wait for those loads counts the
// younger stores: memory instructions of a wavefront finish in order.) us a launch, a workgroup per tile -> walking: 65 536 x
// 1024 -> 4096 609 -> 570, 4096 -> 1024 507 -> 498; 40 000 x 816 -> 2552 225 -> 201; 16 384 x 512 -> 2048 51 -> 43; 30 000 x
// 256 -> 1024 38 -> 29.
template <typename T, int BM, int BN, int WM, int WN, int NST, bool WALK>
__device__ __forceinline__ void gemm_body(const GemmParams& p, unsigned char* const smem, int launch, const int step, const int mx, const int ny) {
  constexpr int KE = 16 / (int)sizeof(T);   // elements per 16-byte chunk
  constexpr int NW = WM * WN;
  constexpr int TM = BM / (32 * WM), TN = BN / (32 * WN);
  constexpr int A_LD = BM / (8 * NW), B_LD = BN / (8 * NW), LPS = A_LD + B_LD;   // load instructions per wavefront and stage
  constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
  static_assert(A_LD >= 1 && B_LD >= 1 && (NST - 2) * LPS < 64 && NST >= 2, "tile shape");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wn = wave / WM;
  int m0, co0;
  const int row_bytes = p.K * (int)sizeof(T), w_bytes = p.k_pad * (int)sizeof(T);
  const int ns = w_bytes / 128;

  // ---- what this lane fetches: row lane / 8 of the 8-row groups wave, wave + NW, ..., chunk
  // (lane & 7) ^ (row / 2 mod 8)
  const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.x), 0, (int)(unsigned)((size_t)p.N * p.x_rows * p.W * row_bytes), 0x00020000);
  const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.w), 0, 0x7fffffff, 0x00020000);
  const int chunk = (lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7);
  static_assert(NW % 2 == 0, "a wavefront's groups have one parity");
  unsigned a_off[A_LD], b_off[B_LD];
  auto set_tile = [&](int at) __attribute__((always_inline)) {
    const TileId tile = xcd_tile_of(at, mx, ny, 1, p.by_group);
    m0 = tile.m * BM; co0 = tile.n * BN;
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int m = m0 + (wave + NW * i) * 8 + (lane >> 3);
      const bool ok = m < p.M;
      const int mm = ok ? m : 0;
      const int q = fastdiv(mm, p.by_w), ow = mm - q * p.W_out;
      const int n = fastdiv(q, p.by_r), r = q - n * p.R;
      const int ih = (p.out_lo + r) * p.sh - p.ph, iw = ow * p.sw - p.pw;
      const bool in = ok & (ih >= p.x_row0) & (ih < p.x_row0 + p.x_rows) & (iw >= 0) & (iw < p.W);
      a_off[i] = in ? (unsigned)(((n * p.x_rows + ih - p.x_row0) * p.W + iw) * row_bytes + chunk * 16) : kOutside;
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) b_off[i] = (unsigned)((co0 + (wave + NW * i) * 8 + (lane >> 3)) * w_bytes + chunk * 16);
  };
  // the chunk lies past the end of the reduction in the last stage
  const bool past = (ns - 1) * 128 + chunk * 16 >= row_bytes;
  auto issue = [&](int s, int j) __attribute__((always_inline)) {   // load instruction j of stage s
    unsigned char* const dst = smem + (s % NST) * STAGE;
    if (j < A_LD) {
      const unsigned off = past & (s == ns - 1) ? kOutside : a_off[j];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (__attribute__((address_space(3))) void*)(dst + (wave + NW * j) * 1024), 16,
                                               (int)off, s * 128, 0, 0);
    } else {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          wbuf, (__attribute__((address_space(3))) void*)(dst + A_BYTES + (wave + NW * (j - A_LD)) * 1024), 16, (int)b_off[j - A_LD],
          s * 128, 0, 0);
    }
  };

  f32x16 acc[TN][TM];

  // ---- fragments: row lane & 31 of a 32-row tile, chunk 2 ks + (lane >> 5); two sets, one being
  // multiplied while the other is read
  const int frow = lane & 31, key = (frow >> 1) & 7;
  const unsigned lds0 = (unsigned)(unsigned long)(__attribute__((address_space(3))) unsigned char*)smem;
  const unsigned a_at = lds0 + (unsigned)(wm * TM * 4096 + frow * 128), b_at = lds0 + (unsigned)(A_BYTES + wn * TN * 4096 + frow * 128);
  u32x4 fa[2][TM], fb[2][TN];
  auto read = [&](int s, int ks, u32x4 (&a)[TM], u32x4 (&b)[TN]) __attribute__((always_inline)) {
    const unsigned off = (unsigned)((s % NST) * STAGE) + (unsigned)(((2 * ks + (lane >> 5)) ^ key) * 16);
    const unsigned aa = a_at + off, bb = b_at + off;
#pragma unroll
    for (int i = 0; i < TN; ++i) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(b[i]) : "v"(bb), "n"(i * 4096) : "memory");
#pragma unroll
    for (int i = 0; i < TM; ++i) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(a[i]) : "v"(aa), "n"(i * 4096) : "memory");
  };
  auto wait_reads = [&](u32x4 (&a)[TM], u32x4 (&b)[TN]) __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(a[i]));
#pragma unroll
    for (int i = 0; i < TN; ++i) asm volatile("" : "+v"(b[i]));
    __builtin_amdgcn_sched_barrier(0);
  };
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  auto multiply = [&](u32x4 (&a)[TM], u32x4 (&b)[TN], int s, bool loads) __attribute__((always_inline)) {
    constexpr int NT = TM * TN, NM = NT * kMmaParts<T>;
#pragma unroll
    for (int i = 0; i < (NM > LPS ? NM : LPS); ++i) {
      if (i < NM) {
        const int t = i % NT;
        mma_part<T>(b[t / TM], a[t % TM], acc[t / TM][t % TM], i / NT);
        if (loads) __builtin_amdgcn_sched_barrier(0);
      }
      if (loads && i < LPS) {
        issue(s, i);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // One stage: four 32-byte steps. (Steps 0..3 use the fragment sets 0, 1, 0, 1.)
  auto stage = [&](int s, bool next, bool refill) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) {
      read(s, ks + 1, fa[(ks + 1) & 1], fb[(ks + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      multiply(fa[ks & 1], fb[ks & 1], 0, false);
      wait_reads(fa[(ks + 1) & 1], fb[(ks + 1) & 1]);
    }
    if (next) {
      if (refill) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 2) * LPS));
      else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      barrier();
      read(s + 1, 0, fa[0], fb[0]);
      __builtin_amdgcn_sched_barrier(0);
    }
    multiply(fa[1], fb[1], s + NST, refill);
    if (next) wait_reads(fa[0], fb[0]);
  };
  auto start = [&]() __attribute__((always_inline)) {   // a tile's first loads
    for (int s = 0; s < NST; ++s)
      if (s < ns)
#pragma unroll
        for (int j = 0; j < LPS; ++j) issue(s, j);
  };
  set_tile(launch);
  start();
  bool behind_stores = false;   // STORES stores are younger than those loads
  constexpr int STORES = TM * TN * 2;
  static_assert(!WALK || (NST - 1) * LPS + STORES < 64, "the counter's range");
  for (;;) {
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
      for (int b = 0; b < TM; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
    if (ns < NST) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    else if (WALK && behind_stores) __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 1) * LPS + STORES));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 1) * LPS));
    barrier();
    read(0, 0, fa[0], fb[0]);
    wait_reads(fa[0], fb[0]);
    int s = 0;
    for (; s + NST < ns; ++s) stage(s, true, true);
    for (; s + 1 < ns; ++s) stage(s, true, false);
    if constexpr (!WALK) {
      stage(s, false, false);
      __syncthreads();
      gemm_epilogue<T, TM, TN>(p, smem, acc, m0, co0, wave, wm, wn, lane);
      return;
    } else {
      const int m_first = m0 + wm * TM * 32, co_first = co0 + wn * TN * 32;
      // (ahead of the next tile's loads: a wait for these is then none for those)
      f32x4 bias[TN][4];
#pragma unroll
      for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          bias[t][g] = p.bias ? *(const f32x4*)(p.bias + min(co_first + t * 32 + g * 8 + (lane >> 5) * 4, p.C_out - 4)) : f32x4{0.f, 0.f, 0.f, 0.f};
      stage(s, false, false);
#pragma unroll
      for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) asm volatile("" : "+v"(bias[t][g]));
      launch += step;
      const bool more = launch < mx * ny;
      behind_stores = m0 + BM <= p.M && co0 + BN <= p.C_out;
      if (more) {
        barrier();   // (no wavefront reads the last stages any more)
        set_tile(launch);
        start();
      }
      gemm_store<T, TM, TN>(p, acc, bias, m_first, co_first, lane);
      if (!more) return;
    }
  }
}

// (The tiles that leave room for one workgroup per compute unit only are walked over.)
template <typename T, int BM, int BN, int WM, int WN, int NST>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2))) void conv_gemm_kernel(const GemmParams p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[gemm_smem<BM, BN, WM, WN, NST>()];
  if constexpr (BM >= 192) {
    if (p.mx) return gemm_body<T, BM, BN, WM, WN, NST, true>(p, smem, blockIdx.x, gridDim.x, p.mx, p.ny);
  }
  gemm_body<T, BM, BN, WM, WN, NST, false>(p, smem, blockIdx.x + gridDim.x * blockIdx.y, 0, gridDim.x, gridDim.y);
}
// The same for several bands of one layer in one grid (band b owns blocks first[b] .. first[b + 1] of x).
template <typename T, int BM, int BN, int WM, int WN, int NST>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2))) void conv_gemm_kernel_bands(const Batch<GemmParams> t) {
  const int b = batch_find(t, blockIdx.x), mx = t.first[b + 1] - t.first[b];
  __shared__ __attribute__((aligned(1024))) unsigned char smem[gemm_smem<BM, BN, WM, WN, NST>()];
  gemm_body<T, BM, BN, WM, WN, NST, false>(t.p[b], smem, (int)blockIdx.x - t.first[b] + mx * (int)blockIdx.y, 0, mx, gridDim.y);
}

// fp32 products on the bf16 matrix cores, which are 16 times as fast as the fp32 ones. A value is the sum of
// three bf16 values (24 bits of mantissa are 8 + 8 + 8, split_bf16), a product of two values the sum of the
// six largest partial products (a published method: Henry, Tang and Heinecke, Leveraging the bfloat16 datatype for
// higher-precision computations, 2019); bf16 products are exact in fp32, and the five small
// partial products have an accumulator of their own. The three dropped ones add up to 2^-24 of the product at most and to 2^-27.5
// typically, so that a sum of a single product is off by up to two roundings of 2^-24 where the fp32 instructions round once;
// a sum of many is closer to 64 bits than theirs, which they round after every second product: rel. error over reductions of 64 / 576 /
// 4608 normal x uniform values 1.5e-7 / 4.3e-7 / 1.2e-6 there, 4.7e-8 / 1.3e-7 / 4.1e-7 here.
// An infinity, a NaN or a value that rounds to infinity in bf16 leaves a sum that is not finite; a workgroup
// that ends with one computes its tile again on the fp32 instructions, every wavefront its part of the reduction, and they
// give what they always did. us a launch without such sums, with one tile of them, with all: 3001 x 512 -> 2048 45 / 82 / 105 (on the fp32
// instructions 55), 2048 -> 512 46 / 125 / 126 (69), 256 x 512 -> 2048 8.8 / 17 / 17 (10.8).
//
//  - The input is split once per workgroup, on its way from memory through registers to LDS: stages of 32
//    elements a row, loaded four stages ahead; a row takes 13 16-byte slots, an odd number, so that 16 neighbouring rows'
//    reads touch every bank once. The weights are split when the plan is made and come straight from memory in
//    operand order, two stages ahead; no two wavefronts load the same ones: a stage's 32 KB take the
//    vector cache 550 cycles (60 bytes a cycle) beside 768 of matrix instructions a SIMD, of the 1 100 it lasts (with 2 x 2 instead
//    of 1 x 4 wavefronts 870 instead of 757 us on 8192 x 1024 -> 4096 -> 1024).
//  - Half of the wavefronts take the first 16 elements of every stage, half the others: a tile is done in half
//    the time where there are few of them, and the sums are added at the end through LDS.
//  - A stage's fragments are read from LDS during the stage before it, the next but one stage's input is split and
//    stored between the matrix instructions.
template <int BM, int BN, int WM, int WN>
__device__ __forceinline__ void gemm_split_body(const GemmParams& p, const int bx, const int gx) {
  constexpr int NW = WM * WN, TM = BM / (32 * WM), TN = BN / (32 * WN);   // NW wavefronts for each step of a stage
  constexpr int PIECES = BM * 8 / (128 * NW);   // 16-byte pieces of a stage's input per lane
  constexpr int PITCH = 208, BUF = BM * PITCH;
  constexpr int SUMS = NW * TM * 4096;          // the other half's sums of one of TN channel tiles
  constexpr int OUT = NW * 32 * gemm_pitch(TN) * 4;
  constexpr int SMEM = 2 * BUF > SUMS ? (2 * BUF > OUT ? 2 * BUF : OUT) : (SUMS > OUT ? SUMS : OUT);
  static_assert(PIECES >= 1, "tile shape");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];
  __shared__ int any_odd;
  if (threadIdx.x == 0) any_odd = 0;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int step = wave / NW, wm = wave % NW % WM, wn = wave % NW / WM;   // this wavefront's step of every stage, and its part of the tile
  const TileId tile = xcd_tile(bx, gx, gridDim.y, 1, p.by_group);
  const int m0 = tile.m * BM, co0 = tile.n * BN;
  const int row_bytes = p.K * 4, ns = p.k_pad / 32;
  const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.x), 0, (int)(unsigned)((size_t)p.N * p.x_rows * p.W * row_bytes), 0x00020000);
  auto pixel_offset = [&](int m) -> unsigned {   // of a pixel's first channel, or outside
    const bool ok = m < p.M;
    const int mm = ok ? m : 0;
    const int q = fastdiv(mm, p.by_w), ow = mm - q * p.W_out;
    const int n = fastdiv(q, p.by_r), r = q - n * p.R;
    const int ih = (p.out_lo + r) * p.sh - p.ph, iw = ow * p.sw - p.pw;
    const bool in = ok & (ih >= p.x_row0) & (ih < p.x_row0 + p.x_rows) & (iw >= 0) & (iw < p.W);
    return in ? (unsigned)(((n * p.x_rows + ih - p.x_row0) * p.W + iw) * row_bytes) : kOutside;
  };
  // ---- this lane's pieces of a stage: four elements from 4 c4 on of row tid / 8 + 16 NW i
  const int c4 = threadIdx.x & 7;
  unsigned src[PIECES];
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    const unsigned at = pixel_offset(m0 + (int)(threadIdx.x >> 3) + i * 16 * NW);
    src[i] = at == kOutside ? kOutside : at + c4 * 16;
  }
  const bool past = (ns - 1) * 128 + c4 * 16 >= row_bytes;   // the piece lies past the end of the reduction in the last stage
  u32x4 raw[2][PIECES];                                      // of the next two stages
  // (Loads are issued for stages past the last one, too, from outside the buffer or of the last weights again: a
  // load under a condition would make every wait one for all loads in flight.)
  auto fetch = [&](int s, u32x4 (&d)[PIECES]) __attribute__((always_inline)) {
    const bool out = (past & (s == ns - 1)) | (s >= ns);
#pragma unroll
    for (int i = 0; i < PIECES; ++i) d[i] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)(out ? kOutside : src[i]), s * 128, 0);
  };
  // [row][step][part][half] x 16 bytes
  unsigned char* const put = smem + (threadIdx.x >> 3) * PITCH + (c4 >> 2) * 96 + ((c4 >> 1) & 1) * 16 + (c4 & 1) * 8;
  auto store = [&](int buf, int i, u32x4 (&d)[PIECES]) __attribute__((always_inline)) {
    uint2 parts[3];
    split_bf16(__builtin_bit_cast(f32x4, d[i]), parts);
#pragma unroll
    for (int k = 0; k < 3; ++k) *(uint2*)(put + buf * BUF + i * 16 * NW * PITCH + k * 32) = parts[k];
  };
  // ---- the weights: [32 channels][step of 16][part][lane] x 16 bytes
  const u32x4* wsrc[TN];
#pragma unroll
  for (int t = 0; t < TN; ++t) wsrc[t] = (const u32x4*)p.w3 + ((size_t)(co0 / 32 + wn * TN + t) * (2 * ns) + step) * 192 + lane;
  u32x4 w[2][TN][3];
  auto fetch_weights = [&](int s, u32x4 (&d)[TN][3]) __attribute__((always_inline)) {
    const int at = min(s, ns - 1) * 384;
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int k = 0; k < 3; ++k) d[t][k] = wsrc[t][(size_t)(at + k * 64)];
  };

  f32x16 acc[TN][TM], low[TN][TM];
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = low[a][b][i] = 0.f;

  const unsigned char* const get = smem + (wm * TM * 32 + (lane & 31)) * PITCH + step * 96 + (lane >> 5) * 16;
  auto read = [&](int buf, u32x4 (&d)[TM][3]) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int b = 0; b < TM; ++b) d[b][k] = *(const u32x4*)(get + buf * BUF + b * 32 * PITCH + k * 32);
  };
  auto barrier = [&]() __attribute__((always_inline)) {   // (for LDS only: loads from memory stay in flight)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  fetch(0, raw[0]);
  fetch_weights(0, w[0]);
  fetch(1, raw[1]);
  fetch_weights(1, w[1]);
#pragma unroll
  for (int set = 0; set < 2; ++set) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i) store(set, i, raw[set]);
    fetch(set + 2, raw[set]);
  }
  u32x4 x[2][TM][3];
  barrier();
  read(0, x[0]);
  // One stage (even ones set 0): its products. Meanwhile the next stage's fragments come out of LDS, and the
  // input of the stage behind that goes into the memory this stage's fragments were read from before the barrier.
  auto stage = [&](int s, int set) __attribute__((always_inline)) {
    barrier();
    read(set ^ 1, x[set ^ 1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      mma_split_part<TN, TM>(w[set], x[set], acc, low, e);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = e * PIECES / 6; i < (e + 1) * PIECES / 6; ++i) store(set, i, raw[set]);
      __builtin_amdgcn_sched_barrier(0);
    }
    fetch(s + 4, raw[set]);
    fetch_weights(s + 2, w[set]);
  };
  int s = 0;
  for (; s + 1 < ns; s += 2) {
    stage(s, 0);
    stage(s + 1, 1);
  }
  if (s < ns) stage(s, 0);

  // ---- sums that are not finite: the workgroup's halves of the reduction once more, on the fp32 instructions
#pragma unroll
  for (int a = 0; a < TN; ++a) {
#pragma unroll
    for (int b = 0; b < TM; ++b) acc[a][b] = (acc[a][b] + low[a][b]) * kSplitUnscale;
    if (any_not_finite(acc[a])) any_odd = 1;
  }
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(any_odd)) {
    unsigned from[TM];
    const u32x4* wrow[TN];
#pragma unroll
    for (int b = 0; b < TM; ++b) from[b] = pixel_offset(m0 + (wm * TM + b) * 32 + (lane & 31));
#pragma unroll
    for (int a = 0; a < TN; ++a) {
      wrow[a] = (const u32x4*)p.w + ((size_t)(co0 / 32 + wn * TN + a) * (p.k_pad / 8) + step * 2) * 64 + lane;
#pragma unroll
      for (int b = 0; b < TM; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
    }
#pragma unroll 2
    for (int i = 0; i < ns; ++i) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int k = i * 32 + step * 16 + j * 8 + (lane >> 5) * 4;
        u32x4 wv[TN];
#pragma unroll
        for (int a = 0; a < TN; ++a) wv[a] = wrow[a][(size_t)(i * 4 + j) * 64];
#pragma unroll
        for (int b = 0; b < TM; ++b) {
          const u32x4 xv = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)((from[b] == kOutside) | (k >= p.K) ? kOutside : from[b] + k * 4), 0, 0);
#pragma unroll
          for (int a = 0; a < TN; ++a) mma<float>(wv[a], xv, acc[a][b]);
        }
      }
    }
  }

  // ---- the two halves of the reduction: the second half's wavefronts hand their sums over through LDS
#pragma unroll
  for (int a = 0; a < TN; ++a) {
    f32x4* const at = (f32x4*)smem + (wave % NW) * TM * 256 + lane;
    if (a > 0) __syncthreads();
    if (step == 1) {
#pragma unroll
      for (int b = 0; b < TM; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) at[(b * 4 + g) * 64] = f32x4{acc[a][b][g * 4], acc[a][b][g * 4 + 1], acc[a][b][g * 4 + 2], acc[a][b][g * 4 + 3]};
    }
    __syncthreads();
    if (step == 0) {
#pragma unroll
      for (int b = 0; b < TM; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 v = at[(b * 4 + g) * 64];
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[a][b][g * 4 + i] += v[i];
        }
    }
  }
  __syncthreads();
  if (step == 1) return;
  gemm_epilogue<float, TM, TN>(p, smem, acc, m0, co0, wave, wm, wn, lane);
}

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(128 * WM * WN) __attribute__((amdgpu_waves_per_eu(2))) void conv_gemm_split_kernel(const GemmParams p) {
  gemm_split_body<BM, BN, WM, WN>(p, blockIdx.x, gridDim.x);
}
// The same for several bands of one layer in one grid (band b owns blocks first[b] .. first[b + 1] of x).
template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(128 * WM * WN) __attribute__((amdgpu_waves_per_eu(2))) void conv_gemm_split_kernel_bands(const Batch<GemmParams> t) {
  const int b = batch_find(t, blockIdx.x);
  gemm_split_body<BM, BN, WM, WN>(t.p[b], blockIdx.x - t.first[b], t.first[b + 1] - t.first[b]);
}

// [c_out_pad][k_pad] fp32 -> [c_out_pad / 32][k_pad / 16][part][half*32 + c_out % 32] x 8 elements
__global__ __launch_bounds__(256) void split_weights_kernel(const float* w, int k_pad, unsigned pieces, u32x4* w3) {
  const unsigned i = blockIdx.x * 256 + threadIdx.x;
  if (i >= pieces) return;
  const unsigned lane = i & 63, steps = (unsigned)k_pad / 16, step = (i >> 6) % steps, group = (i >> 6) / steps;
  const float* const from = w + (size_t)(group * 32 + (lane & 31)) * k_pad + step * 16 + (lane >> 5) * 8;
  uint2 lo[3], hi[3];
  split_bf16(*(const f32x4*)from, lo);
  split_bf16(*(const f32x4*)(from + 4), hi);
#pragma unroll
  for (int k = 0; k < 3; ++k) w3[(size_t)(i >> 6) * 192 + k * 64 + lane] = u32x4{lo[k].x, lo[k].y, hi[k].x, hi[k].y};
}

GemmParams make_gemm(const OpLaunch& L) {
  GemmParams p;
  p.x = L.x.ptr; p.y = L.y.ptr; p.y2 = L.y2; p.res = L.res.ptr; p.w = L.w; p.w3 = L.w3; p.bias = L.bias;
  p.x_row0 = L.x.row0; p.x_rows = L.x.rows; p.W = L.x.w; p.K = L.x.c;
  p.y_row0 = L.y.row0; p.y_rows = L.y.rows; p.W_out = L.y.w; p.C_out = L.y.c;
  p.r_row0 = L.res.row0; p.r_rows = L.res.rows;
  p.sh = L.sh; p.sw = L.sw; p.ph = L.ph; p.pw = L.pw; p.act = L.act; p.k_pad = L.k_pad;
  p.out_lo = L.out_lo; p.R = L.out_hi - L.out_lo; p.N = L.x.n;
  p.M = p.N * p.R * p.W_out; p.mx = p.ny = 0;
  p.by_w = make_fastdiv(p.W_out); p.by_r = make_fastdiv(p.R); p.by_group = make_fastdiv(1);
  return p;
}

bool gemm_shape(const OpLaunch& L) {
  const int esz = L.dtype == LOP_BF16 ? 2 : 4, ke = 16 / esz;
  if (L.op != LOP_CONV2D || L.kh != 1 || L.kw != 1 || L.x.c % ke != 0 || L.y.c % ke != 0) return false;
  if (L.x.c * esz < 256) return false;                                    // (at least two stages)
  if ((size_t)L.k_pad * esz * conv_cout_pad(L.y.c) >= ((size_t)1 << 31)) return false;
  return (size_t)L.x.n * L.x.rows * L.x.w * L.x.c * esz < ((size_t)1 << 31);
}

// Workgroups of a launch of 256 x 256 or 192 x 256 tiles: one per compute unit, each of which walks over its share of the tiles (and, the
// number being a multiple of the XCDs, over tiles of the XCD it runs on).
constexpr long kWalkers = 256;

// The tile of a launch over the bands of a group, or bm == 0 where there is too little of it for these
// tiles and the mid-size kernels, which split the reduction over the wavefronts, are faster.
// Measured, in us before -> after: bf16 8192 x 1024 -> 4096 (512 tiles of 256 x 256) 94 -> 76 (68 walking), 8192 x 4096 ->
// 1024 (128 of them) 88 -> 93 alone but 1 396 -> 1 059 for both layers on four streams, since only the
// 256-wide tile asks the L2s for little enough while other launches run beside it; 5422 x 984 -> 1040
// (215 tiles of 128 x 256) 31 -> 24; 4096 x 4096 -> 1024 (512 of 128 x 64) 89 -> 43, against 53 with 128 tiles
// of 128 x 256; 1000 x 2048 -> 512 (64 of 128 x 64) 11 there, 16 here. fp32 on its own instructions, reductions of 64 to 191
// elements: mid-size kernels / 64 x 64 / 128 x 128 tiles, K 64 and 188: 3001 x K -> 256 (188 tiles of 64 x 64) 5.0 / 5.2 / 11.8 and 9.0 / 7.5 /
// 19.5, 1500 -> 1024 (384) 7.8 / 7.0 / 12.2 and 13.2 / 11.4 / 19.9, 1000 -> 512 (128) 4.2 / 5.0 / 11.6 and 8.4 / 7.0 / 19.1; 20000 -> 512
// (628 tiles of 128 x 128) 29.4 / 23.2 / 29.0 and 56 / 43.7 / 50.6, 8000 -> 2048 (1 008) 36.9 / 35.1 / 33.8 and 71.6 / 63.6 / 63.1, 8000 -> 3000 (1 512) 51.2 /
// 48.9 / 47.8 and 104 / 87.7 / 92.1, 16000 -> 2048 (2 000) 66.1 / 63.1 / 62.4 and 137 / 119 / 121.
struct GemmChoice { int bm = 0, bn = 0; bool split = false; };
constexpr long kBigTiles = 128;        // 256 x 256, bf16
// 192 x 256, bf16, in place of 256 x 256 in a chain on a caller's stream where the last of several rounds of those would be at most
// a third full and whole rounds of the smaller, which take 0.8 of the time each, cost less. us a call of one layer there, eight
// buffers in turn (more than the caches hold), 256 -> 192: 9 116 x 1024 -> 2048 (288 -> 384 tiles) 58.1 -> 49.9, 22 940 x 512 -> 600 (270 ->
// 360) 39.4 -> 32.9, 20 380 x 1024 -> 1024 (320 -> 428) 60.2 -> 59.6, 44 956 x 1000 -> 600 (528 -> 705) 98.0 -> 90.2, 67 484 x 512 -> 512 (528 -> 704)
// 62.7 -> 61.6, 36 252 x 512 -> 512 (284 -> 378), bound by memory, 40.7 -> 40.8; with a residual 9 116 x 2048 -> 2048 112.1 -> 93.9, 36 252 x
// 512 -> 512 50.3 -> 47.2; in four bands of 134 x 134 pixels 256 -> 1024 channels behind 64 -> 256 (3 x 3) 40.8 -> 35.8. With other chains beside it a
// nearly empty round is no loss, they fill it, and the smaller tile reads more for a product: two layers in flight 65 792 x 512 -> 512 ->
// 512 108.2 -> 114.9, 34 816 x 512 -> 1024 -> 512 96.4 -> 101.6, 25 000 x 768 -> 3072 -> 768 258 -> 266, 9 000 x 512 -> 2048 -> 512
// 59.2 -> 58.2. With half a last round there is nothing to gain (24 000 x 1000 -> 2000 -> 1000, 376 -> 500, 230 -> 231). A single round is left to
// the larger tile (65 536 x 1024 -> 4096 -> 1024 in eight bands on four streams 1 008 -> 1 068), and so are reductions of more than 3 072
// (20 000 x 4096 -> 1024 gains 2 %). Nothing stops the rule at 256
// elements but that it was found there: 9 000 x 128 -> 2048 -> 128 40.2 -> 37.1, 33 000 x 192 -> 512 -> 192 47.6 -> 44.2.
constexpr double kLessTile = 0.8;
constexpr int kLessMinK = 256, kLessMaxK = 3072;
constexpr long kWideTiles = 192;       // 128 x 256, bf16
constexpr long kNarrowTiles = 384;     // 128 x 64, bf16
constexpr long kF32BigTiles = 1024;    // 128 x 128, fp32
constexpr long kF32Tiles = 320;        // 64 x 64, fp32
// 64 x 128, fp32 on the bf16 matrix cores. Before -> here, us a launch: 3001 x 512 -> 2048 (752 tiles) 64 -> 45, 2048 -> 512 (188)
// 69 -> 45, 1500 x 1024 -> 512 (96) 24.1 -> 23.5, 600 x 512 -> 2048 (160) 22.0 -> 16.1; one stage after the other they
// take 0.55 us a stage whatever runs beside them. Short reductions have nothing to gain: 3001 x 128 -> 256 7.0 -> 8.9.
// 32 x 64 of them, four times as many: a stage takes 0.3 us, so few tiles are faster alone, but four of them take more of the
// chip from other launches than the one. Alone, before / 64 x 128 / 32 x 64, and in flight: 256 x 512 -> 2048 (256 of them) 10.8 / 14.7 / 8.9, 7.6 / 5.1 /
// 4.7; 1000 x 2048 -> 512 (256) 32.4 / 39.0 / 27.8, 25.9 / 13.5 / 14.8; 300 x 512 -> 2048 (320) 13.8 / 14.9 / 10.5, 9.5 / 5.8 / 5.6; 600 x
// 1024 -> 1024 (304) 23.6 / 23.2 / 17.2, 16.5 / 8.6 / 9.3; 1100 x 2048 -> 512 (280) 42.3 / 39.4 / 29.9, 27.9 / 14.5 / 16.1. So they are
// taken where there is at most one to a compute unit, and with short reductions, where they lose nothing in flight, as far
// as the larger ones are slower alone than what was there before. Fewer yet are left to the mid-size kernels, which
// split the reduction: 128 x 512 -> 2048 (128 of 32 x 64) 7.5 there, 8.3 here, 300 x 2048 -> 512 (80) 20.5 and 25.3.
constexpr long kSplitTiles = 64;
constexpr int kSplitMinK = 192;
constexpr long kSplitSmallTiles = 256;                     // 32 x 64
constexpr long kSplitShortTiles = 96;                      // 64 x 128, with reductions of at most
constexpr int kSplitShortK = 512;

GemmChoice choose_gemm(const OpLaunch* Ls, int n) {
  for (int b = 0; b < n; ++b)
    if (!gemm_shape(Ls[b])) return {};
  const int c_out = Ls[0].y.c;
  auto tiles = [&](int bm, int bn) {
    if ((c_out + bn - 1) / bn * bn > conv_cout_pad(c_out)) return 0L;
    long t = 0;
    for (int b = 0; b < n; ++b) t += ((long)Ls[b].x.n * std::max(Ls[b].out_hi - Ls[b].out_lo, 0) * Ls[b].y.w + bm - 1) / bm;
    return t * ((c_out + bn - 1) / bn);
  };
  if (Ls[0].dtype == LOP_BF16) {
    if (const long t = tiles(256, 256); t >= kBigTiles) {
      auto rounds = [](long n) { return (double)((n + kWalkers - 1) / kWalkers); };
      const long last = t % kWalkers;
      const bool thin = Ls[0].alone && Ls[0].x.c >= kLessMinK && Ls[0].x.c <= kLessMaxK && t > kWalkers && last > 0 && 3 * last <= kWalkers;
      return thin && rounds(tiles(192, 256)) * kLessTile < rounds(t) ? GemmChoice{192, 256} : GemmChoice{256, 256};
    }
    if (tiles(128, 64) < kNarrowTiles) return {};
    return tiles(128, 256) >= kWideTiles ? GemmChoice{128, 256} : GemmChoice{128, 64};
  }
  if (const long t = Ls[0].w3 ? tiles(64, 128) : 0; t >= kSplitTiles) {
    const bool small = tiles(32, 64) <= kSplitSmallTiles || (t < kSplitShortTiles && Ls[0].x.c <= kSplitShortK);
    return small ? GemmChoice{32, 64, true} : GemmChoice{64, 128, true};
  }
  if (tiles(128, 128) >= kF32BigTiles) return {128, 128};
  return tiles(64, 64) >= kF32Tiles ? GemmChoice{64, 64} : GemmChoice{};
}

// Whether a launch of 256 x 256 or 192 x 256 tiles walks. Not with a residual: its loads would wait for the next tile's, which are older (17 497 x
// 504 -> 888 behind 888 -> 504, chains in flight: 53.5 us a call if both walk, 47.1 if the first does, 49.0 if none). Nor with a second destination, of
// the size that has one a launch has no second round.
bool walks(const GemmParams& p) { return !p.res && !p.y2; }

// single, bands: a kernel of BM x BN tiles and THREADS threads, for one band and for several; PARTS: of products made of parts
template <int BM, int BN, int THREADS, bool PARTS = false>
hipError_t launch_tile(void (*single)(const GemmParams), void (*bands)(const Batch<GemmParams>), const OpLaunch* Ls, int n, hipStream_t s,
                       KernelEvents* ev) {
  GemmParams ps[kMaxBatch];
  unsigned gx[kMaxBatch];
  const unsigned gy = (unsigned)((Ls[0].y.c + BN - 1) / BN);
  if ((int)gy * BN > conv_cout_pad(Ls[0].y.c)) return hipErrorInvalidValue;  // unguarded weight loads
  int m = 0;
  for (int b = 0; b < n; ++b) {
    ps[m] = make_gemm(Ls[b]);
    if (ps[m].M <= 0) continue;
    if (PARTS) ps[m].w = Ls[b].wd;
    ps[m].by_group = make_fastdiv(kGroupM * (int)gy);
    gx[m] = (unsigned)((ps[m].M + BM - 1) / BM);
    ++m;
  }
  if (m == 0) return hipSuccess;
  if (BM >= 192 && m == 1 && walks(ps[0])) {
    ps[0].mx = (int)gx[0]; ps[0].ny = (int)gy;
    const long tiles = (long)gx[0] * gy;
    return launch_kernel(single, dim3((unsigned)std::min(tiles, kWalkers)), dim3(THREADS), s, ev, ps[0]);
  }
  return launch_group(single, bands, ps, m, gx, gy, 1, dim3(THREADS), s, ev);
}
template <typename T, int BM, int BN, int WM, int WN, int NST>
hipError_t launch_direct(const OpLaunch* Ls, int n, hipStream_t s, KernelEvents* ev) {
  return launch_tile<BM, BN, 64 * WM * WN>(conv_gemm_kernel<T, BM, BN, WM, WN, NST>, conv_gemm_kernel_bands<T, BM, BN, WM, WN, NST>, Ls, n, s, ev);
}
template <int BM, int BN, int WM, int WN>
hipError_t launch_split(const OpLaunch* Ls, int n, hipStream_t s, KernelEvents* ev) {
  return launch_tile<BM, BN, 128 * WM * WN, true>(conv_gemm_split_kernel<BM, BN, WM, WN>, conv_gemm_split_kernel_bands<BM, BN, WM, WN>, Ls, n, s, ev);
}

}  // namespace

bool split_shape(int c_in, int kh, int kw, int sh, int sw, int dilation) {
  if (kh == 1 && kw == 1) return c_in >= kSplitMinK;
  return kh == 3 && kw == 3 && c_in % 32 == 0 && sh == sw && sh <= 2 && dilation == 1;   // (the patch form's, see patch_shape)
}
hipError_t launch_split_weights(const void* w, int c_out_pad, int k_pad, void* w3, hipStream_t stream) {
  const unsigned pieces = (unsigned)((size_t)c_out_pad * k_pad / 8);
  return launch_kernel(split_weights_kernel, dim3((pieces + 255) / 256), dim3(256), stream, nullptr, (const float*)w, k_pad, pieces, (u32x4*)w3);
}

bool gemm_applies(const OpLaunch* Ls, int n) { return n >= 1 && n <= kMaxBatch && choose_gemm(Ls, n).bm != 0; }

hipError_t launch_gemm(const OpLaunch* Ls, int n, hipStream_t s, KernelEvents* ev) {
  if (n < 1 || n > kMaxBatch) return hipErrorInvalidValue;
  const GemmChoice c = choose_gemm(Ls, n);
  if (Ls[0].dtype == LOP_BF16) {
    if (c.bm == 256) return launch_direct<__bf16, 256, 256, 2, 4, 2>(Ls, n, s, ev);
    if (c.bm == 192) return launch_direct<__bf16, 192, 256, 2, 4, 2>(Ls, n, s, ev);
    if (c.bm == 128 && c.bn == 256) return launch_direct<__bf16, 128, 256, 2, 4, 3>(Ls, n, s, ev);
    if (c.bm == 128) return launch_direct<__bf16, 128, 64, 2, 2, 3>(Ls, n, s, ev);
    return hipErrorInvalidValue;
  }
  if (c.split) return c.bm == 32 ? launch_split<32, 64, 1, 2>(Ls, n, s, ev) : launch_split<64, 128, 1, 4>(Ls, n, s, ev);
  if (c.bm == 128) return launch_direct<float, 128, 128, 2, 2, 2>(Ls, n, s, ev);
  if (c.bm == 64) return launch_direct<float, 64, 64, 2, 2, 3>(Ls, n, s, ev);
  return hipErrorInvalidValue;
}

int gemm_describe(const OpLaunch* Ls, int n, char* name, size_t size) {
  const GemmChoice c = choose_gemm(Ls, n);
  const bool bf = Ls[0].dtype == LOP_BF16;
  int m = 0;
  for (int b = 0; b < n; ++b) m += make_gemm(Ls[b]).M > 0;
  if (name && size && c.split)
    snprintf(name, size, "conv_gemm_split_kernel%s<%d, %d, 1, %d>", m > 1 ? "_bands" : "", c.bm, c.bn, c.bn / 32);
  else if (name && size)   // (tile, wavefronts in either direction, stages: as launch_gemm takes them)
    snprintf(name, size, "conv_gemm_kernel%s<%s, %d, %d, 2, %d, %d>", m > 1 ? "_bands" : "", bf ? "__bf16" : "float", c.bm, c.bn,
             bf && c.bn == 256 ? 4 : 2, c.bm >= 192 || (!bf && c.bm == 128) ? 2 : 3);
  return 1;
}

}  // namespace lop
