// Dense 3 x 3 convolution on a row interval, the LDS-staged kernel in its patch form.
//
// conv_lds_kernel of conv_igemm.hip fetches every tap of every pixel of its tile: nine times the
// input under a 3 x 3 filter, and what the L2s and the load path deliver of that (16 to 29 bytes per
// clock and compute unit observed) is what bounds it. Here a workgroup owns a rectangle of output pixels x BN
// channels and fetches the input pixels under that rectangle once per 128 bytes of channels (a
// "patch": 180 pixels for 8 x 16 outputs, 1.4 x the outputs instead of 9 x); all nine taps are then
// read from LDS at offsets from each other. The filter is not staged at all: it comes straight
// from memory in MFMA operand order (OpLaunch::wd), a contiguous KiB per wavefront load, nine taps
// ahead of its use.
//
//  - The four wavefronts split the reduction inside a patch (wavefront w multiplies the w-th 32
//    bytes of every pixel) and each accumulates the whole tile, so that no filter byte is loaded
//    twice by a workgroup and no barrier is needed between taps: one per 128 bytes of channels,
//    where the next patch, fetched meanwhile, takes over. Their partial tiles are added through
//    LDS in wavefront order. (Tiles of 128 x 64: halves instead of quarters, see patch_wide_body.)
//  - A pixel of the patch takes 144 bytes of LDS: with an odd number of 16-byte slots per pixel the
//    16 lanes that read a slot of 16 neighbouring pixels at a time touch every bank once, and a tap is
//    a constant number of bytes away from another. (global -> LDS loads fill consecutive slots, so
//    every ninth lane of them fetches nothing.)
//  - The input slab is a buffer resource: a pixel outside the image or the slab is a load past its
//    end, which puts zeros into LDS without touching memory.
//  - S == 2: the patch keeps the even and the odd columns of a row apart, so that neighbouring
//    output pixels read neighbouring slots there, too.
//  - POOL: the 2 x 2 stride-2 max pooling behind the convolution is part of the launch. The lanes take
//    the tile's pixels window by window, so that a window is four neighbouring lanes of the summed
//    tile: the maximum is taken between them before bias, activation and rounding (all of them
//    non-decreasing) and the convolution's own output never exists in memory.
//
// (What it is worth, measured: see choose_patch. fp32 has a form of its own: patch_split_body.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>

#include "act.hpp"
#include "conv_common.hpp"
#include "conv_split.hpp"
#include "conv_tiles.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

constexpr int kPixelBytes = 144, kPixelSlots = 9;

// Row and column, inside the tile, of its pixel i.
template <bool POOL>
__device__ __forceinline__ void tile_pixel(const PatchParams& p, int i, int& r, int& c) {
  if constexpr (POOL) {
    const int v = i >> 2, vr = smalldiv(v, p.by_tw), vc = v - vr * (p.tw >> 1);   // (by_tw divides by tw / 2)
    r = vr * 2 + ((i >> 1) & 1);
    c = vc * 2 + (i & 1);
  } else {
    r = smalldiv(i, p.by_tw);
    c = i - r * p.tw;
  }
}

// Where a workgroup's tile lies: its first row of the launch and first column, its image and its channel tile;
// second: a channel tile of the 1 x 1 convolution beside the launch's own.
struct PatchAt { int n, r0, c0, tile_n; bool second; };
__device__ __forceinline__ PatchAt patch_at(const PatchParams& p, int bx, int gx, bool siblings) {
  const TileId tile = xcd_tile(bx, gx, gridDim.y, 1, p.by_group);
  PatchAt a;
  a.second = siblings && tile.n >= p.sib.first;
  a.tile_n = a.second ? tile.n - p.sib.first : tile.n;
  const int q = fastdiv(tile.m, p.by_ntx), tx = tile.m - q * p.ntx;
  a.n = fastdiv(q, p.by_nty);
  a.r0 = (q - a.n * p.nty) * p.th;
  a.c0 = tx * p.tw;
  return a;
}

// What follows the sums of N pieces of one fragment (32 pixels; piece i: channels first + 8 i ..): pooling, bias,
// residual, activation, the one rounding. load issues everything that has to come from memory.
template <typename T, int N, bool POOL>
struct PatchPieces {
  typedef unsigned raw_t __attribute__((ext_vector_type(sizeof(T))));   // four elements
  f32x4 bias[N];
  raw_t res[N];
  int row, col, first;
  bool live;

  __device__ __forceinline__ void load(const PatchParams& p, const PatchAt& t, int fragment, int first_channel, int lane) {
    const int half = lane >> 5, C_out = t.second ? p.sib.C_out : p.C_out;
    const float* const bias_at = t.second ? p.sib.bias : p.bias;
    first = first_channel;
    int r, c;
    tile_pixel<POOL>(p, fragment * 32 + (lane & 31), r, c);
    row = t.r0 + r;
    col = t.c0 + c;
    live = (r < p.th) & (row < p.R) & (col < p.Wc);
    if (t.second) live = live & (p.out_lo + row >= p.sib.lo) & (p.out_lo + row < p.sib.hi);
#pragma unroll
    for (int i = 0; i < N; ++i) bias[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (bias_at) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int co = first + i * 8 + half * 4;
        bias[i] = *(const f32x4*)(bias_at + (co < C_out ? co : 0));
      }
    }
    if constexpr (!POOL) {
      if (p.res && !t.second) {
        const size_t ra = live ? ((size_t)(t.n * p.r_rows + p.out_lo + row - p.r_row0) * p.W_out + col) * p.C_out : 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const int co = first + i * 8 + half * 4;
          res[i] = *(const raw_t*)((const T*)p.res + ra + (co < p.C_out ? co : 0));
        }
      } else {
#pragma unroll
        for (int i = 0; i < N; ++i) res[i] = raw_t(0u);
      }
    }
  }

  __device__ __forceinline__ void store(const PatchParams& p, const PatchAt& t, f32x4 (&sum)[N], int lane) {
    const int half = lane >> 5, C_out = t.second ? p.sib.C_out : p.C_out;
    const Clamp cl = make_clamp(t.second ? p.sib.act : p.act);
    T* const y = (T*)(t.second ? p.sib.y : p.y);
    T* const y2 = t.second ? nullptr : (T*)p.y2;
    size_t ya;
    bool stores = live;
    if constexpr (POOL) {
#pragma unroll
      for (int i = 0; i < N; ++i) max_of_quad(sum[i], bias[i]);
      stores = live & ((lane & 3) == 0);
      ya = ((size_t)(t.n * p.y_rows + ((p.out_lo + row) >> 1) - p.y_row0) * p.W_out + (col >> 1)) * p.C_out;
    } else {
      ya = ((size_t)(t.n * (t.second ? p.sib.y_rows : p.y_rows) + p.out_lo + row - (t.second ? p.sib.y_row0 : p.y_row0)) * p.W_out + col) * C_out;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if constexpr (!POOL) {
        sum[i] += bias[i];
        alignas(16) T rr[4];
        *(raw_t*)rr = res[i];
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[i][j] += to_f32(rr[j]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) sum[i][j] = clamp_act(sum[i][j], cl);
    }
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int co = first + i * 8 + half * 4;
        if (stores && co < C_out) {
          *(f32x4*)(y + ya + co) = sum[i];
          if (y2) *(f32x4*)(y2 + ya + co) = sum[i];
        }
      }
    } else {
      auto pack = [&](int i) {
        alignas(8) __bf16 o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = (__bf16)sum[i][j];
        return *(const uint2*)o;
      };
      if constexpr (N == 1) {
        const uint2 o = pack(0);
        const int co = first + half * 4;
        if (stores && co < C_out) {
          *(uint2*)(y + ya + co) = o;
          if (y2) *(uint2*)(y2 + ya + co) = o;
        }
      } else {
        // two pieces hold 16 channels of a pixel in two lanes, 4 + 4 interleaved: exchanged between
        // the lane halves so that each ends with 8 consecutive ones (one 16-byte store)
#pragma unroll
        for (int i = 0; i < N; i += 2) {
          const uint2 e = pack(i), o = pack(i + 1);
          const auto s0 = __builtin_amdgcn_permlane32_swap(e.x, o.x, false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(e.y, o.y, false, false);
          const u32x4 v = u32x4{(unsigned)s0[0], (unsigned)s1[0], (unsigned)s0[1], (unsigned)s1[1]};
          const int co = first + i * 8 + half * 8;
          if (stores && co < C_out) {
            *(u32x4*)(y + ya + co) = v;
            if (y2) *(u32x4*)(y2 + ya + co) = v;
          }
        }
      }
    }
  }
};

// The four partial tiles, added in wavefront order through LDS, and what follows the sums. again(acc): this wavefront's
// partial tile once more, in fp32 for a workgroup that has a sum that is not finite (any_odd: zero in LDS since a barrier).
template <typename T, int TP, bool POOL, typename Again>
__device__ __forceinline__ void patch_finish(const PatchParams& p, unsigned char* smem, f32x16 (&acc)[TP], const PatchAt& t,
                                             int lane, int wave, int* any_odd, Again&& again) {
  // wavefront w finishes pieces w TP .. (w + 1) TP of the UNITS (32 pixels x 8 channels) pieces of a tile (piece u:
  // fragment u / 4, channels (u % 4) * 8 ..), which all lie in one fragment
  constexpr int UNITS = TP * 4;
  u32x4* const part = (u32x4*)smem;
  PatchPieces<T, TP, POOL> out;
  out.load(p, t, wave * TP / 4, t.tile_n * 32 + ((wave * TP) & 3) * 8, lane);
  if constexpr (sizeof(T) == 4) {
    if (any_not_finite(acc)) *any_odd = 1;
  }
  __syncthreads();
  if constexpr (sizeof(T) == 4) {
    if (__builtin_amdgcn_readfirstlane(*any_odd)) again(acc);
  }
#pragma unroll
  for (int u = 0; u < UNITS; ++u) {
    const f32x16& s = acc[u / 4];
    const int g = (u % 4) * 4;
    part[(wave * UNITS + u) * 64 + lane] = __builtin_bit_cast(u32x4, f32x4{s[g], s[g + 1], s[g + 2], s[g + 3]});
  }
  __syncthreads();
  f32x4 sum[TP];
#pragma unroll
  for (int i = 0; i < TP; ++i) {
    sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) sum[i] += __builtin_bit_cast(f32x4, part[(s * UNITS + wave * TP + i) * 64 + lane]);
  }
  out.store(p, t, sum, lane);
}

// Where the pixels of a patch lie in the input slab. What a workgroup works out before its first load is issued is
// waited for by all of it, and with few wavefronts on a compute unit an instruction takes about five cycles, a product of 32 bits
// about twenty: all products here are of 24 bits (the slab has less than 2^24 pixels of 128 bytes or more, see patch_shape).
// 206 instructions in front of the first load became 140; with the same in the walking and the narrow kernel (370 became 40
// and 150 about 115) chains take, us alone: detector encoder in 16 bands 279 -> 273, bf16 stack in 8 bands 222 -> 217, fp32
// backbone with shared rows 146 -> 140 (in flight 80.7 -> 78.5 beside other streams).
template <int S>
struct PatchWindow {
  int row, rows, col, base;   // first row and column, rows of the patch up to the slab's end; row 0 of the image
  __device__ __forceinline__ PatchWindow(const PatchParams& p, const PatchAt& t) {
    row = (p.out_lo + t.r0) * S - p.ph - p.x_row0;
    rows = min(p.x_rows, row + p.ph_rows);
    col = t.c0 * S - p.pw;
    base = t.n * p.x_rows;
  }
  // `bytes` into the patch's pixel `pix`, or outside
  __device__ __forceinline__ unsigned at(const PatchParams& p, int pix, int row_bytes, int bytes) const {
    const int pr = smalldiv(pix, p.by_pitch), pc = pix - (int)__umul24(pr, p.pitch), half_cols = p.pitch >> 1;
    const int ih = row + pr, iw = col + (S == 1 ? pc : (pc < half_cols ? 2 * pc : 2 * (pc - half_cols) + 1));
    const unsigned px = __umul24(base + ih, p.W) + iw, to = __umul24(px, row_bytes) + bytes;
    return (ih >= 0) & (ih < rows) & ((unsigned)iw < (unsigned)p.W) ? to : kOutside;
  }
};

// The slots of a patch that this lane fetches (16 bytes each; the ninth of every nine slots, and what lies outside the
// patch, the slab or the image, is a load past the buffer's end).
template <int NI, int S>
__device__ __forceinline__ void patch_slots(const PatchParams& p, const PatchAt& t, int wave, int lane, unsigned (&src)[NI], int row_bytes) {
  const PatchWindow<S> win(p, t);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int slot = (i * 4 + wave) * 64 + lane;
    const int pix = smalldiv(slot, small_div(kPixelSlots)), k = slot - pix * kPixelSlots;
    const unsigned at = win.at(p, pix, row_bytes, k * 16);
    src[i] = k < 8 ? at : kOutside;
  }
}

// TP x 32 pixels x 32 channels per workgroup; NI: load instructions per wavefront and patch.
template <typename T, int TP, int NI, bool POOL, int S>
__device__ __forceinline__ void patch_body(const PatchParams& p, const int bx, const int gx) {
  constexpr int KE = 16 / (int)sizeof(T), NT = 1;
  constexpr int BUF = NI * 4096;            // bytes of a patch in LDS
  constexpr int SMEM = 2 * BUF > TP * 16384 ? 2 * BUF : TP * 16384;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int px = lane & 31, half = lane >> 5;
  const PatchAt tile = patch_at(p, bx, gx, S == 2);
  const bool second = tile.second;
  const int tile_n = tile.tile_n;
  const int row_bytes = p.C_in * (int)sizeof(T);
  const int chunks = row_bytes / 128;

  const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.x), 0, (int)((size_t)p.N * p.x_rows * p.W * row_bytes), 0x00020000);
  unsigned src[NI];
  patch_slots<NI, S>(p, tile, wave, lane, src, row_bytes);
  auto fetch_patch = [&](int c) __attribute__((always_inline)) {
    unsigned char* const dst = smem + (c & 1) * BUF;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (__attribute__((address_space(3))) void*)(dst + (i * 4 + wave) * 1024),
                                               16, (int)src[i], c * 128, 0, 0);
    // (the filter loads behind these stay behind them: the waits below count on that order)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // ---- the filter: [32 channels][step][lane] 16 bytes; this wavefront's step of a tap and patch
  const u32x4* wsrc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
    wsrc[t] = (const u32x4*)(second ? p.sib.wd : p.wd) + ((size_t)(tile_n * NT + t) * (second ? p.sib.k_steps : p.k_steps) + wave) * 64 + lane;
  const int tap_steps = p.C_in / (2 * KE) * 64;
  u32x4 wreg[9][NT];
  auto fetch_tap = [&](int c, int t) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NT; ++k) wreg[t][k] = wsrc[k][(size_t)(t * tap_steps + c * 256)];
  };

  fetch_patch(0);
  if (!second) {
#pragma unroll
    for (int t = 0; t < 9; ++t) fetch_tap(0, t);
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  // ---- this lane's pixel of every 32-pixel fragment: row and column inside the tile, and where the
  // first tap of it lies in a patch
  int at[TP];
  const unsigned lds0 = (unsigned)(unsigned long)(__attribute__((address_space(3))) unsigned char*)smem;
#pragma unroll
  for (int f = 0; f < TP; ++f) {
    int r, c;
    tile_pixel<POOL>(p, f * 32 + px, r, c);
    r = min(r, p.th - 1);                   // (lanes past the tile compute its last row again; they store nothing)
    at[f] = (int)lds0 + ((r * S) * p.pitch + c) * kPixelBytes + wave * 32 + half * 16;
  }
  const int tap_row = p.pitch * kPixelBytes;
  const int tap_odd = S == 1 ? kPixelBytes : (p.pitch >> 1) * kPixelBytes;

  f32x16 acc[NT][TP];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < TP; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

  // Pixel fragments are read with instructions of our own: reads the compiler can see would make
  // it wait for every load in flight to LDS.
  u32x4 pa[TP], pb[TP];
  auto read_tap = [&](int buf, int t, u32x4 (&d)[TP]) __attribute__((always_inline)) {
    const int a = t / 3, b = t % 3;
    const int off = buf + a * tap_row + (S == 2 && b == 1 ? tap_odd : 0);
    constexpr int step = S == 1 ? kPixelBytes : kPixelBytes / 2;   // (S == 2: two taps further is the next even column)
#pragma unroll
    for (int f = 0; f < TP; ++f) {
      const int addr = at[f] + off;
      if (b == 0 || (S == 2 && b == 1)) asm volatile("ds_read_b128 %0, %1" : "=v"(d[f]) : "v"(addr) : "memory");
      else if (b == 1) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d[f]) : "v"(addr), "n"(step) : "memory");
      else asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d[f]) : "v"(addr), "n"(2 * step) : "memory");
    }
  };
  auto wait_reads = [&](u32x4 (&d)[TP]) __attribute__((always_inline)) {
    if constexpr (TP == 4) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]), "+v"(d[3]) :: "memory");
    else if constexpr (TP == 2) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(d[0]), "+v"(d[1]) :: "memory");
    else { static_assert(TP == 1, "tiles of 32, 64 or 128 pixels"); asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(d[0]) :: "memory"); }
  };
  // One patch: nine taps, the fragments of the next tap on their way while one is multiplied; MORE:
  // another patch follows, a tap's filter registers are refilled for it as soon as they are free.
  auto run_patch = [&](int c, bool more) __attribute__((always_inline)) {
    const int buf = (c & 1) * BUF;
    read_tap(buf, 0, pa);
    wait_reads(pa);
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      u32x4 (&now)[TP] = (t & 1) ? pb : pa;
      u32x4 (&nxt)[TP] = (t & 1) ? pa : pb;
      if (t < 8) read_tap(buf, t + 1, nxt);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < kMmaParts<T>; ++e)
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
          for (int f = 0; f < TP; ++f) mma_part<T>(wreg[t][a], now[f], acc[a][f], e);
      __builtin_amdgcn_sched_barrier(0);
      if (more) fetch_tap(c + 1, t);
      __builtin_amdgcn_sched_barrier(0);
      if (t < 8) wait_reads(nxt);
    }
  };
  auto patch_barrier = [&]() __attribute__((always_inline)) {
    // this wavefront's part of the patch has arrived: only the nine taps' filter loads are younger
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(9 * NT));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  if (second) {   // one tap, the centre
    for (int c = 0; c < chunks; ++c) {
      u32x4 w1[NT];
#pragma unroll
      for (int k = 0; k < NT; ++k) w1[k] = wsrc[k][(size_t)(c * 256)];
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (c + 1 < chunks) fetch_patch(c + 1);
      read_tap((c & 1) * BUF, 4, pa);
      wait_reads(pa);
#pragma unroll
      for (int e = 0; e < kMmaParts<T>; ++e)
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
          for (int f = 0; f < TP; ++f) mma_part<T>(w1[a], pa[f], acc[a][f], e);
    }
  } else {
    int c = 0;
    for (; c + 1 < chunks; ++c) {
      patch_barrier();
      fetch_patch(c + 1);      // (into the buffer every wavefront was done with at the barrier)
      run_patch(c, true);
    }
    patch_barrier();
    run_patch(c, false);
  }

  patch_finish<T, TP, POOL>(p, smem, acc[0], tile, lane, wave, nullptr, [](f32x16 (&)[TP]) {});
}

// The 128 x 64 tile (bf16): two wavefronts to a half of the channels, each with half of every pixel's 128 bytes.
// Against four wavefronts that take a quarter of the pixels' bytes for the whole tile, the same filter vectors and twice the
// reads from LDS (128 of the 240 bytes it serves per cycle, when the matrix cores are busy all the time), but a quarter of
// the partial sums (32 KB instead of 128 through LDS, one exchange instead of two) and half the accumulators, which
// took the register file to its end and four vectors of every tile to memory. Four
// quarters took 28.7 us for 256 -> 256 channels on 14 300 pixels (0.59 PFLOP/s), this 21.4; pooled, 512 -> 512 on 3 136,
// 25 and 20.3.
template <int NI, bool POOL>
__device__ __forceinline__ void patch_wide_body(const PatchParams& p, const int bx, const int gx) {
  typedef __bf16 T;
  constexpr int TP = 4, BUF = NI * 4096, STEPS = 18;   // half steps of a patch: 9 taps x 2
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * BUF];
  static_assert(2 * BUF >= 4 * 8192, "the exchange of partial sums");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int px = lane & 31, half = lane >> 5, part = wave & 1;
  const PatchAt tile = patch_at(p, bx, gx, false);
  const int row_bytes = p.C_in * 2, chunks = row_bytes / 128;
  const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.x), 0, (int)((size_t)p.N * p.x_rows * p.W * row_bytes), 0x00020000);
  unsigned src[NI];
  patch_slots<NI, 1>(p, tile, wave, lane, src, row_bytes);
  auto fetch_patch = [&](int c) __attribute__((always_inline)) {
    unsigned char* const dst = smem + (c & 1) * BUF;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (__attribute__((address_space(3))) void*)(dst + (i * 4 + wave) * 1024),
                                               16, (int)src[i], c * 128, 0, 0);
    // (the filter loads behind these stay behind them: the waits below count on that order)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  fetch_patch(0);
  // ---- the filter: [32 channels][step][lane] 16 bytes; this wavefront's two steps of a tap and patch
  const int co0 = tile.tile_n * 64 + (wave >> 1) * 32;
  const u32x4* const wsrc = (const u32x4*)p.wd + ((size_t)(co0 / 32) * p.k_steps + 2 * part) * 64 + lane;
  const int tap_steps = p.C_in / 16 * 64;
  u32x4 wreg[STEPS];
  auto fetch_tap = [&](int c, int t) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 2; ++k) wreg[2 * t + k] = wsrc[(size_t)(t * tap_steps + c * 256 + k * 64)];
  };
#pragma unroll
  for (int t = 0; t < 9; ++t) fetch_tap(0, t);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  // ---- this lane's pixel of every 32-pixel fragment: where the first tap of it lies in a patch
  int at[TP];
  const unsigned lds0 = (unsigned)(unsigned long)(__attribute__((address_space(3))) unsigned char*)smem;
#pragma unroll
  for (int f = 0; f < TP; ++f) {
    int r, c;
    tile_pixel<POOL>(p, f * 32 + px, r, c);
    r = min(r, p.th - 1);                   // (lanes past the tile compute its last row again; they store nothing)
    at[f] = (int)lds0 + (r * p.pitch + c) * kPixelBytes + part * 64 + half * 16;
  }
  const int tap_row = p.pitch * kPixelBytes;
  f32x16 acc[TP];
#pragma unroll
  for (int f = 0; f < TP; ++f)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[f][i] = 0.f;

  // Pixel fragments are read with instructions of our own (reads the compiler can see would make it wait for every
  // load in flight to LDS), two half steps ahead of their products.
  u32x4 frag[3][TP];
  auto read = [&](int buf, auto index, u32x4 (&d)[TP]) __attribute__((always_inline)) {
    constexpr int i = decltype(index)::value, t = i / 2, off = t % 3 * kPixelBytes + i % 2 * 32;
    const int row = buf + t / 3 * tap_row;
#pragma unroll
    for (int f = 0; f < TP; ++f) {
      const int addr = at[f] + row;
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d[f]) : "v"(addr), "n"(off) : "memory");
    }
  };
  auto wait_reads = [&](auto younger, u32x4 (&d)[TP]) __attribute__((always_inline)) {
    constexpr int n = decltype(younger)::value;
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]), "+v"(d[3]) : "n"(n) : "memory");
  };
  // One patch; more: another follows, a tap's filter registers are refilled for it as soon as they are free.
  auto run_patch = [&](int c, bool more) __attribute__((always_inline)) {
    const int buf = (c & 1) * BUF;
    read(buf, std::integral_constant<int, 0>{}, frag[0]);
    read(buf, std::integral_constant<int, 1>{}, frag[1]);
    unroll<STEPS>([&](auto index) __attribute__((always_inline)) {
      constexpr int i = decltype(index)::value;
      if constexpr (i + 2 < STEPS) read(buf, std::integral_constant<int, (i + 2) % STEPS>{}, frag[(i + 2) % 3]);
      wait_reads(std::integral_constant<int, i + 2 < STEPS ? 2 * TP : i + 1 < STEPS ? TP : 0>{}, frag[i % 3]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int f = 0; f < TP; ++f) mma<T>(wreg[i], frag[i % 3][f], acc[f]);
      __builtin_amdgcn_sched_barrier(0);
      if (i % 2 == 1 && more) fetch_tap(c + 1, i / 2);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto patch_barrier = [&]() __attribute__((always_inline)) {
    // this wavefront's part of the patch has arrived: only the nine taps' filter loads are younger
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(STEPS));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  int c = 0;
  for (; c + 1 < chunks; ++c) {
    patch_barrier();
    fetch_patch(c + 1);      // (into the buffer every wavefront was done with at the barrier)
    run_patch(c, true);
  }
  patch_barrier();
  run_patch(c, false);

  // ---- a wavefront finishes fragments 2 part and 2 part + 1: it hands the others' sums to its neighbour
  PatchPieces<T, 4, POOL> out[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) out[k].load(p, tile, 2 * part + k, co0, lane);
  f32x4* const mine = (f32x4*)smem + wave * 512 + lane, * const theirs = (f32x4*)smem + (wave ^ 1) * 512 + lane;
  __syncthreads();
  auto pick = [&](int k, int g, bool second) __attribute__((always_inline)) {   // (selected by value: acc stays in registers)
    f32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = second ? acc[2 + k][g * 4 + j] : acc[k][g * 4 + j];
    return v;
  };
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int g = 0; g < 4; ++g) mine[(k * 4 + g) * 64] = pick(k, g, part == 0);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    f32x4 sum[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) sum[g] = pick(k, g, part == 1) + theirs[(k * 4 + g) * 64];
    out[k].store(p, tile, sum, lane);
  }
}

// The fp32 form: products on the bf16 matrix cores (conv_gemm.hip says how, and how precise). A pixel of the patch is
// split into its three bf16 parts on the way from memory through registers to LDS, 208 bytes for 32 channels
// (an odd number of 16-byte slots again); the filter's parts are made with the plan and loaded a patch ahead. Of the 18 steps of 16
// channels that a patch has per pixel, wavefronts 0 and 2 take the first 16 channels and 1 and 3 the second, 0 and 1 five taps
// and 2 and 3 four of an even patch, the other way round of an odd one. A patch is 864 TP cycles of matrix instructions
// (2 304 TP on the fp32 ones), 300 to 700 of vector instructions and about 1 100 of loads (65 KB at the vector
// cache's 60 bytes a cycle), shared by the two or three workgroups of a compute unit; alone it takes 1 800 (TP = 1) or 2 900.
// Wavefronts that split the filter themselves load 4 bytes a weight instead of 6, but their vector instructions
// (1 150 + 150 TP cycles, without scaling) bounded it: us a launch, then and now, 128 -> 128 channels on 784 pixels 8.1 and 6.6,
// 256 -> 256 on 400 12.7 and 9.6, on 1 600 18.2 and 16.0; the fp32 backbone in flight 121.7 and 119.2, with shared rows 55.6 and 55.2,
// alone 154 and 145.
// A workgroup with a sum that is not finite computes its tile again on the fp32 instructions, a quarter of the reduction a
// wavefront: us a launch without such sums, with one tile of them, with all: 128 -> 128 channels on 784 pixels 6.6 / 15 / 16 (on the fp32
// instructions 7.7), 256 -> 256 on 1 600 16 / 41 / 49 (22), 512 -> 512 on 196 16 / 48 / 48 (23).
template <int TP, int NI, bool POOL, int S>
__device__ __forceinline__ void patch_split_body(const PatchParams& p, const int bx, const int gx) {
  constexpr int PB = 208, BUF = NI * 32 * PB;
  constexpr int SMEM = 2 * BUF > TP * 16384 ? 2 * BUF : TP * 16384;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];
  __shared__ int any_odd;
  if (threadIdx.x == 0) any_odd = 0;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int px = lane & 31, half = lane >> 5, step = wave & 1;
  const PatchAt tile = patch_at(p, bx, gx, S == 2);
  const bool second = tile.second;
  const int row_bytes = p.C_in * 4, chunks = p.C_in / 32;
  const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.x), 0, (int)((size_t)p.N * p.x_rows * p.W * row_bytes), 0x00020000);
  const int ih0 = (p.out_lo + tile.r0) * S - p.ph, iw0 = tile.c0 * S - p.pw;
  auto input = [&](int ih, int iw) -> unsigned {   // of a pixel's first channel, or outside
    const bool ok = (ih >= p.x_row0) & (ih < p.x_row0 + p.x_rows) & (iw >= 0) & (iw < p.W);
    return ok ? (unsigned)(((tile.n * p.x_rows + ih - p.x_row0) * p.W + iw) * row_bytes) : kOutside;
  };
  // ---- the pieces this lane moves of every patch: channels 4 k .. 4 k + 3 of pixel threadIdx.x / 8 + 32 i
  const int k4 = threadIdx.x & 7;
  const PatchWindow<S> win(p, tile);
  unsigned src[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int pix = i * 32 + (int)(threadIdx.x >> 3);
    src[i] = win.at(p, pix, row_bytes, k4 * 16);
  }
  u32x4 raw[2][NI];   // of the next two patches
  // (Loads are issued for patches past the last one, too, from outside the buffer or of the last filter again: a
  // load under a condition would make every wait one for all loads in flight.)
  auto fetch_patch = [&](int c, u32x4 (&d)[NI]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
      d[i] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)(c < chunks ? src[i] : kOutside), c * 128, 0);
  };
  unsigned char* const put = smem + (threadIdx.x >> 3) * PB + (k4 >> 2) * 96 + (k4 >> 1 & 1) * 16 + (k4 & 1) * 8;
  auto store = [&](int buf, int i, u32x4 (&d)[NI]) __attribute__((always_inline)) {
    uint2 parts[3];
    split_bf16(__builtin_bit_cast(f32x4, d[i]), parts);
#pragma unroll
    for (int k = 0; k < 3; ++k) *(uint2*)(put + buf * BUF + i * 32 * PB + k * 32) = parts[k];
  };
  // ---- the filter: five taps (four, and one of them twice) of a patch, three parts of 16 channels each, and the tap that
  // is being multiplied (so that its registers are free for the next patch's filter a tap earlier)
  const u32x4* const w3 = (const u32x4*)p.w3 + (size_t)tile.tile_n * (p.k_steps / 2) * 192 + lane;
  auto first_tap = [&](int c) { return (wave >> 1 ^ c) & 1 ? 5 : 0; };
  u32x4 w[5][3], tap[2][1][3];
  auto fetch_tap = [&](int c, int j) __attribute__((always_inline)) {
    const int cc = min(c, chunks - 1);
    const u32x4* const from = w3 + (size_t)((min(first_tap(cc) + j, 8) * (p.C_in / 16) + cc * 2 + step) * 192);
#pragma unroll
    for (int k = 0; k < 3; ++k) w[j][k] = from[k * 64];
  };
  auto take_tap = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 3; ++k) tap[j & 1][0][k] = w[j][k];
  };
  // ... and the fp32 values, 32 channels' pieces of four elements a step
  const u32x4* const wd = (const u32x4*)(second ? p.sib.wd : p.wd) + (size_t)tile.tile_n * (second ? p.sib.k_steps : p.k_steps) * 64;

  fetch_patch(0, raw[0]);
  if (!second) {
#pragma unroll
    for (int j = 0; j < 5; ++j) fetch_tap(0, j);
  }
  fetch_patch(1, raw[1]);

  // ---- this lane's pixel of every 32-pixel fragment: where the first tap of it lies in a patch
  int at[TP];
#pragma unroll
  for (int f = 0; f < TP; ++f) {
    int r, c;
    tile_pixel<POOL>(p, f * 32 + px, r, c);
    r = min(r, p.th - 1);                   // (lanes past the tile compute its last row again; they store nothing)
    at[f] = ((r * S) * p.pitch + c) * PB + step * 96 + half * 16;
  }
  f32x16 acc[1][TP], low[1][TP];
#pragma unroll
  for (int f = 0; f < TP; ++f)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[0][f][i] = low[0][f][i] = 0.f;

  auto read_tap = [&](int buf, int t, u32x4 (&d)[TP][3]) __attribute__((always_inline)) {
    const int a = t >= 6 ? 2 : t >= 3 ? 1 : 0, b = t - 3 * a;
    // (S == 2: an odd column lies half a row further, two columns further is the next even one)
    const int off = buf + (a * p.pitch + (S == 1 ? b : b == 1 ? p.pitch >> 1 : b >> 1)) * PB;
#pragma unroll
    for (int f = 0; f < TP; ++f)
#pragma unroll
      for (int k = 0; k < 3; ++k) d[f][k] = *(const u32x4*)(smem + at[f] + off + k * 32);
  };
#pragma unroll
  for (int i = 0; i < NI; ++i) store(0, i, raw[0]);
  fetch_patch(2, raw[0]);
  u32x4 x[2][TP][3];
  auto barrier = [&]() __attribute__((always_inline)) {   // (for LDS only: loads from memory stay in flight)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto multiply = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 6; ++e) mma_split_part<1, TP>(tap[j & 1], x[j & 1], acc, low, e);
  };
  // One patch (even ones in the first half of LDS, set 0). While a tap is multiplied, the next one's pixels come out of
  // LDS, and the next patch is split and stored into the memory that every wavefront was done with at the barrier: vector
  // instructions between the matrix instructions, which keep their pipe busy for 32 cycles each.
  auto run_patch = [&](int c, int set) __attribute__((always_inline)) {
    barrier();
    const int buf = set * BUF, t0 = first_tap(c);
    read_tap(buf, t0, x[0]);
    take_tap(0);
    fetch_tap(c + 1, 0);
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      if (j < 4) {
        read_tap(buf, min(t0 + j + 1, 8), x[(j + 1) & 1]);
        multiply(j);
        take_tap(j + 1);
        fetch_tap(c + 1, j + 1);
      }
#pragma unroll
      for (int i = j * NI / 5; i < (j + 1) * NI / 5; ++i) store(set ^ 1, i, raw[set ^ 1]);
      if (j < 4) {
#pragma unroll
        for (int i = 0; i < 6 * TP; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix instruction,
          __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);   // eight vector instructions
        }
      }
    }
    fetch_patch(c + 3, raw[set ^ 1]);
    __builtin_amdgcn_sched_barrier(0);
    if (t0 == 0) multiply(4);
  };
  if (second) {   // one tap, the centre, of weights that have no parts: a lane's eight channels are half a step
    for (int c = 0; c < chunks; ++c) {
      const u32x4* const from = wd + (size_t)(c * 4 + 2 * step + half) * 64 + px;
      split_bf16(from[0], from[32], tap[0][0]);
      barrier();
      if (wave < 2) {
        read_tap((c & 1) * BUF, 4, x[0]);
        multiply(0);
      }
      fetch_patch(c + 1, raw[0]);
#pragma unroll
      for (int i = 0; i < NI; ++i) store((c & 1) ^ 1, i, raw[0]);
    }
  } else {
    int c = 0;
    for (; c + 1 < chunks; c += 2) {
      run_patch(c, 0);
      run_patch(c + 1, 1);
    }
    if (c < chunks) run_patch(c, 0);
  }
#pragma unroll
  for (int f = 0; f < TP; ++f) acc[0][f] = (acc[0][f] + low[0][f]) * kSplitUnscale;

  // fp32 instructions, on operands straight from memory: every fourth step of 8 channels of all taps
  auto again = [&](f32x16 (&sum)[TP]) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < TP; ++f)
#pragma unroll
      for (int i = 0; i < 16; ++i) sum[f][i] = 0.f;
    for (int t = second ? 4 : 0; t < (second ? 5 : 9); ++t) {
      const u32x4* const wt = wd + (size_t)(second ? 0 : t * (p.C_in / 8)) * 64 + wave * 64 + lane;
      unsigned from[TP];
#pragma unroll
      for (int f = 0; f < TP; ++f) {
        int r, c;
        tile_pixel<POOL>(p, f * 32 + px, r, c);
        const unsigned at = input(ih0 + r * S + t / 3, iw0 + c * S + t % 3);
        from[f] = at == kOutside ? kOutside : at + wave * 32 + half * 16;
      }
#pragma unroll 2
      for (int c = 0; c < chunks; ++c) {
        const u32x4 wv = wt[(size_t)c * 256];
#pragma unroll
        for (int f = 0; f < TP; ++f) mma<float>(wv, __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)from[f], c * 128, 0), sum[f]);
      }
    }
  };
  patch_finish<float, TP, POOL>(p, smem, acc[0], tile, lane, wave, &any_odd, again);
}

// Load instructions per wavefront and patch: the patch of a tile has at most NI * 256 / 9 pixels.
constexpr int patch_loads(int tp, int s) { return s == 1 ? (tp == 4 ? 7 : tp == 2 ? 4 : 3) : 6; }
constexpr int patch_room(int bm, int s) { return patch_loads(bm / 32, s) * 256 / kPixelSlots; }

template <typename T, int BM, int BN, bool POOL, int S>
__device__ __forceinline__ void patch_tile(const PatchParams& p, const int bx, const int gx) {
  if constexpr (sizeof(T) == 4) {
    static_assert(BN == 32, "the fp32 form has one channel tile");
    patch_split_body<BM / 32, patch_loads(BM / 32, S), POOL, S>(p, bx, gx);
  } else if constexpr (BM == 128) {
    static_assert(BN == 64 && S == 1, "the wide form");
    patch_wide_body<patch_loads(4, 1), POOL>(p, bx, gx);
  } else {
    static_assert(BN == 32, "one channel tile");
    patch_body<T, BM / 32, patch_loads(BM / 32, S), POOL, S>(p, bx, gx);
  }
}

template <typename T, int BM, int BN, bool POOL, int S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void conv_patch_kernel(const PatchParams p) {
  patch_tile<T, BM, BN, POOL, S>(p, blockIdx.x, gridDim.x);
}
// The same for several bands of one layer in one grid (band b owns blocks first[b] .. first[b + 1] of x).
template <typename T, int BM, int BN, bool POOL, int S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void conv_patch_kernel_bands(const Batch<PatchParams> t) {
  const int b = batch_find(t, blockIdx.x);
  patch_tile<T, BM, BN, POOL, S>(t.p[b], blockIdx.x - t.first[b], t.first[b + 1] - t.first[b]);
}

bool patch_shape(const OpLaunch& L) {
  const bool bf = L.dtype == LOP_BF16;
  const int esz = bf ? 2 : 4, ke = 16 / esz;
  if (L.op != LOP_CONV2D || !L.wd || L.kh != 3 || L.kw != 3 || L.dh != 1 || L.dw != 1) return false;
  if (L.sh != L.sw || (L.sh != 1 && L.sh != 2)) return false;
  if (L.x.c * esz % 128 != 0 || (size_t)L.x.c * esz >= (1 << 24) || L.y.c % ke != 0 || (!bf && !L.w3)) return false;
  return (size_t)L.x.n * L.x.rows * L.x.w * L.x.c * esz < ((size_t)1 << 31);
}

// The tile of a launch over the bands of a group, or bm == 0 when another kernel is the faster one.
// What a tile costs was fitted to measured launches of the three backbones, one image and all bands
// together (cycles; chunk: 128 bytes of channels): a compute unit that has several tiles to do gets
// through them at `chunk` each plus `rest` per tile (the L2s deliver 16-19 TB/s to the whole chip, which
// a larger tile asks less of per product: 128 -> 128 channels on 12 500 pixels take 8.7 us with
// 128 x 64 tiles and 9.5 with 64 x 32, 256 -> 256 on 6 400 12.9 and 14.5, on 3 100 11.6 and 8.6), and no
// launch is faster than one tile from beginning to end (`first` + `alone` per chunk: 512 -> 512
// channels on 196 pixels 5.6 us with 32 x 32 tiles, 6.5 with 64 x 32, 15.6 with 128 x 64, 16.1 before).
// Pooled, the 128 x 64 tile has to be 15 % ahead: the fit does not know what follows the sums there (64 -> 64 channels
// on 40 300 pixels 9.0 us against 7.7 with 64 x 32, 128 -> 128 on 10 100 7.5 against 6.7). Without pooling it leaves other
// launches more of the chip than the smaller tiles, also where those are faster alone (with such a margin there, too, the 720p
// chain's 16 bands took 157 us instead of 154 with calls in flight).
struct PatchChoice { int bm = 0, bn = 0; };
struct PatchCost { int bm, bn; double chunk, rest, alone, first; };
constexpr PatchCost kBf16Costs[] = {
    {128, 64, 5000, 3500, 3300, 6000}, {64, 32, 1860, 840, 1100, 3500}, {32, 32, 1200, 620, 750, 3000}};
// fp32, fitted alike (chunk: 32 channels); 64 x 32 against 32 x 32 tiles: 64 -> 64 channels on 25 600 pixels 19.3 and 22.0 us,
// on 6 400 7.2 and 7.5, on 3 136 6.9 and 5.3; 256 -> 256 on 3 136 27.3 and 32.1, on 1 600 16.2 and 17.2, on 784 14.4 and 10.5.
constexpr PatchCost kF32Costs[] = {{64, 32, 4150, 4600, 2900, 4700}, {32, 32, 2300, 2700, 1790, 3100}};
constexpr int kPatchUnits = 256;
// fp32 launches of fewer tiles are left to the kernels that cut the reduction finer (16 x 16 tiles, or
// slices across workgroups). At 100 tiles this one is ahead (128 -> 128 channels on 784 pixels: 8.2 us there, 6.6 here;
// 256 -> 256 on 400, 104 tiles: 11.1 and 9.6), and alone it stays so down to about 50 (64 -> 64 on 784, 50 tiles: 7.6 and 5.2; 256 -> 256 on
// 324, 88: 10.8 and 9.4; but 256 -> 512, stride 2, on 144, 80: 11.3 and 11.9); a line at 50 changes the fp32 backbone with
// shared rows by nothing in flight (55.2 and 55.3 us) and alone (144).
constexpr long kF32MinTiles = 100;
// bf16: a handful of compute units cannot stream megabytes of filter (7 x 7 x 512 channels is 32 tiles: 5.6 us
// here, 8.9 there)
constexpr long kBf16MinTiles = 24;
// Stride 2: a patch is four times the outputs, so a tile fetches nearly twice what the kernel that fetches taps does per
// output (2.25 of them) and gains by waiting for them once instead of nine times. fp32 launches always take it (there -> here,
// us alone: 64 -> 128 channels on 3 136 pixels 11.6 -> 9.1). On the fp32 instructions they
// were faster alone where the reduction is short (64 -> 128 on 784 pixels 5.8 against 6.4, on 5 625 12.2 and 13.7; 128 -> 256 on
// 784 8.8 and 8.7), but not with other launches beside them: the fp32 backbone in flight took 131 us instead of 119.6
// with that layer on them, with shared rows 56.7 instead of 55.2 (142 instead of 145 alone). bf16
// ones up to one tile per compute unit: beyond that they are ahead alone up to about four (128 -> 256 on 3 600 pixels, 904
// tiles, 9.6 -> 8.9; on 6 400, 1 600 tiles, 12.3 -> 13.2), but not with other launches beside them (detector encoder with
// shared rows, one launch of 904 tiles: 63.9 -> 64.9 us a chain).
constexpr long kStride2MaxTiles = kPatchUnits;

PatchChoice choose_patch(const OpLaunch* convs, const OpLaunch* pools, int n) {
  const OpLaunch& L = convs[0];
  for (int b = 0; b < n; ++b)
    if (!patch_shape(convs[b])) return {};
  const bool bf = L.dtype == LOP_BF16;
  auto tiles = [&](int bm, int bn) {
    long t = 0;
    for (int b = 0; b < n; ++b) {
      const PatchWork w = patch_work(convs[b], pools ? &pools[b] : nullptr);
      if (w.R <= 0) continue;
      const PatchTile pt = tile_for(w, bm, patch_room(bm, L.sh), L.sh, pools != nullptr);
      if (!pt.th) return 0L;
      t += pt.tiles;
    }
    return t * ((L.y.c + bn - 1) / bn);
  };
  const long small = tiles(32, 32);
  if (small < (bf ? kBf16MinTiles : kF32MinTiles)) return {};
  if (L.sh == 2) return !pools && (!bf || small <= kStride2MaxTiles) ? PatchChoice{32, 32} : PatchChoice{};
  const double chunks = L.x.c * (bf ? 2 : 4) / 128;
  PatchChoice best;
  double best_cost = 0;
  auto weigh = [&](const PatchCost& c) {
    const long t = tiles(c.bm, c.bn);
    if (t == 0) return;
    const double share = (double)t / kPatchUnits;
    const double cost = std::max(share * (chunks * c.chunk + c.rest) + c.first / 2, chunks * c.alone + c.first) * (pools && c.bm == 128 ? 1.15 : 1);
    if (!best.bm || cost < best_cost) { best = {c.bm, c.bn}; best_cost = cost; }
  };
  if (bf) for (const PatchCost& c : kBf16Costs) weigh(c);
  else for (const PatchCost& c : kF32Costs) weigh(c);
  return best;
}

// sibs: per band the 1 x 1 convolution that the launch computes as well, or nullptr
template <typename T, int BM, int BN>
hipError_t launch_tile(const OpLaunch* convs, const OpLaunch* pools, const OpLaunch* sibs, int n, hipStream_t s, KernelEvents* ev) {
  PatchParams ps[kMaxBatch];
  unsigned gx[kMaxBatch];
  const unsigned gy1 = (unsigned)((convs[0].y.c + BN - 1) / BN), gy2 = sibs ? (unsigned)((sibs[0].y.c + BN - 1) / BN) : 0, gy = gy1 + gy2;
  if ((int)gy1 * BN > conv_cout_pad(convs[0].y.c)) return hipErrorInvalidValue;  // unguarded weight loads
  if (sibs && (convs[0].sh != 2 || (int)gy2 * BN > conv_cout_pad(sibs[0].y.c))) return hipErrorInvalidValue;
  int m = 0;
  for (int b = 0; b < n; ++b) {
    const PatchWork w = patch_work(convs[b], pools ? &pools[b] : nullptr);
    if (w.R <= 0) continue;
    ps[m] = make_patch(convs[b], pools ? &pools[b] : nullptr, BM, patch_room(BM, convs[b].sh), gy, &gx[m]);
    if (sibs) {
      const OpLaunch& q = sibs[b];
      ps[m].sib = Sibling{q.wd, q.y.ptr, q.bias, q.k_pad / (32 / (int)sizeof(T)), q.y.row0, q.y.rows, q.y.c, q.act, q.out_lo, q.out_hi, (int)gy1};
    }
    const int room = patch_room(BM, convs[b].sh);
    if (ps[m].th < 1 || ps[m].ph_rows * ps[m].pitch > room || ps[m].th * ps[m].tw > BM) return hipErrorInvalidValue;
    ++m;
  }
  if (m == 0) return hipSuccess;
  if (convs[0].sh == 1) {
    if (pools)
      return launch_group(conv_patch_kernel<T, BM, BN, true, 1>, conv_patch_kernel_bands<T, BM, BN, true, 1>, ps, m, gx, gy, 1,
                          dim3(256), s, ev);
    return launch_group(conv_patch_kernel<T, BM, BN, false, 1>, conv_patch_kernel_bands<T, BM, BN, false, 1>, ps, m, gx, gy, 1,
                        dim3(256), s, ev);
  }
  if constexpr (BM != 32) {
    return hipErrorInvalidValue;
  } else {
    if (pools) return hipErrorInvalidValue;
    return launch_group(conv_patch_kernel<T, BM, BN, false, 2>, conv_patch_kernel_bands<T, BM, BN, false, 2>, ps, m, gx, gy, 1,
                        dim3(256), s, ev);
  }
}

}  // namespace

bool patch_applies(const OpLaunch* convs, const OpLaunch* pools, int n) {
  return n >= 1 && n <= kMaxBatch && choose_patch(convs, pools, n).bm != 0;
}

hipError_t launch_patch(const OpLaunch* convs, const OpLaunch* pools, int n, hipStream_t s, KernelEvents* ev) {
  if (n < 1 || n > kMaxBatch) return hipErrorInvalidValue;
  const PatchChoice c = choose_patch(convs, pools, n);
  if (convs[0].dtype == LOP_BF16) {
    if (c.bm == 128) return launch_tile<__bf16, 128, 64>(convs, pools, nullptr, n, s, ev);
    if (c.bm == 64) return launch_tile<__bf16, 64, 32>(convs, pools, nullptr, n, s, ev);
    if (c.bm == 32) return launch_tile<__bf16, 32, 32>(convs, pools, nullptr, n, s, ev);
    return hipErrorInvalidValue;
  }
  if (c.bm == 64) return launch_tile<float, 64, 32>(convs, pools, nullptr, n, s, ev);
  if (c.bm == 32) return launch_tile<float, 32, 32>(convs, pools, nullptr, n, s, ev);
  return hipErrorInvalidValue;
}

// A 3 x 3 convolution of stride 2 and the 1 x 1 one beside it, where the former takes this kernel.
bool patch_takes_sibling(const OpLaunch* convs, const OpLaunch* sibs, int n) {
  if (n < 1 || n > kMaxBatch || convs[0].sh != 2 || !sibs[0].wd || sibs[0].y.c % (convs[0].dtype == LOP_BF16 ? 8 : 4) != 0) return false;
  return choose_patch(convs, nullptr, n).bm == 32;
}
hipError_t launch_patch_siblings(const OpLaunch* convs, const OpLaunch* sibs, int n, hipStream_t s, KernelEvents* ev) {
  if (!patch_takes_sibling(convs, sibs, n)) return hipErrorInvalidValue;
  return convs[0].dtype == LOP_BF16 ? launch_tile<__bf16, 32, 32>(convs, nullptr, sibs, n, s, ev)
                                    : launch_tile<float, 32, 32>(convs, nullptr, sibs, n, s, ev);
}

int patch_describe(const OpLaunch* convs, const OpLaunch* pools, int n, char* name, size_t size) {
  const PatchChoice c = choose_patch(convs, pools, n);
  int m = 0;
  for (int b = 0; b < n; ++b) m += patch_work(convs[b], pools ? &pools[b] : nullptr).R > 0;
  if (name && size)
    snprintf(name, size, "conv_patch_kernel%s<%s, %d, %d, %s, %d>", m > 1 ? "_bands" : "",
             convs[0].dtype == LOP_BF16 ? "__bf16" : "float", c.bm, c.bn, pools ? "true" : "false", convs[0].sh);
  return 1;
}

}  // namespace lop
