// 3 x 3 convolutions of few input channels at many pixels: the filter stays in registers.
//
// With 32 or 64 bf16 channels in (pixels of 64 or 128 bytes) the reduction is one patch long: the kernels that give
// every workgroup one tile spend it on starting up, on loading the filter and on adding partial
// tiles. Here a wavefront keeps the whole filter of 32 output channels in registers as matrix
// operands (18 or 36 vectors of 16 bytes) and its workgroup walks over tiles of the output: per tile the
// four wavefronts fetch the input pixels under it (a patch) once, straight to LDS, while they
// work on the patch before it, and each multiplies 32 output pixels by its 32 channels over the
// whole reduction - no partial sums, one barrier per tile.
//
//  - WCO of the four wavefronts take different channels of the same pixels: a patch is then shared by
//    32 WCO output channels, and 32 * 4 / WCO pixels are a tile.
//  - LDS: a pixel takes an odd number of 16-byte slots, so that neighbouring pixels' reads touch every
//    bank once; with stride 2 the even columns of a row lie before its odd ones.
//  - A tile's results are stored after the next tile's barrier. The wait before a barrier is for
//    everything in flight (loads and stores share a counter): the patch to come and those stores have
//    then both had a whole tile's products to complete.
//  - Workgroups are as many as are resident at once; XCD k walks the k-th eighth of a band's tiles,
//    neighbouring workgroups on neighbouring tiles, so that halos are found in that XCD's L2.
//
// (What it is worth, measured: see choose_walk.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "act.hpp"
#include "conv_common.hpp"
#include "conv_tiles.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

// PIXB: bytes of an input pixel; S: stride; WCO: blocks of 32 output channels per workgroup
template <int PIXB, int S, int WCO>
struct WalkTile {
  static constexpr int SLOTS = PIXB / 16 + 1, PB = SLOTS * 16;   // 16-byte slots and bytes of a pixel in LDS
  static constexpr int KS = PIXB / 32;                           // reduction steps of a tap
  static constexpr int PIXELS = 128 / WCO;
  static constexpr int NI = S == 1 ? 4 : 6;                      // load instructions per wavefront and patch
  static constexpr int ROOM = NI * 256 / SLOTS;                  // pixels of a patch
  static constexpr int BUF = NI * 4096;
  static constexpr int AHEAD = KS == 2 && S == 1 ? 2 : 1;         // taps read from LDS ahead of the one multiplied (as registers allow)
};

template <int OFF>
__device__ __forceinline__ void lds_read(u32x4& d, int addr) {
  // (reads of our own: those the compiler can see would make it wait for every load in flight to LDS)
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF) : "memory");
}
// The KS reduction steps of tap T of a lane's pixel.
template <int S, int PB, int KS, int T>
__device__ __forceinline__ void read_tap(int here, int tap_row, int tap_odd, u32x4 (&d)[KS]) {
  constexpr int b = T % 3, off = S == 1 ? b * PB : (b == 2 ? PB : 0);
  const int addr = here + T / 3 * tap_row + (S == 2 && b == 1 ? tap_odd : 0);
  lds_read<off>(d[0], addr);
  lds_read<off + 32>(d[1], addr);
  if constexpr (KS == 4) {
    lds_read<off + 64>(d[2], addr);
    lds_read<off + 96>(d[3], addr);
  }
}
template <int N>
__device__ __forceinline__ void wait_reads(u32x4 (&d)[2]) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(d[0]), "+v"(d[1]) : "n"(N) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_reads(u32x4 (&d)[4]) {
  asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]), "+v"(d[3]) : "n"(N) : "memory");
}

template <int PIXB, int S, int WCO, bool POOL>
__device__ __forceinline__ void walk_body(const PatchParams& p, const int bx, const int gx) {
  typedef WalkTile<PIXB, S, WCO> G;
  constexpr int SLOTS = G::SLOTS, PB = G::PB, KS = G::KS, NI = G::NI, BUF = G::BUF, AHEAD = G::AHEAD;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * BUF];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int px = lane & 31, half = lane >> 5;
  const int co0 = (blockIdx.y * WCO + wave % WCO) * 32, frag = wave / WCO;

  // ---- this workgroup's tiles: first, first + step, ... below end
  const int tiles = p.N * p.nty * p.ntx;
  const int xs = (unsigned)gx % kXcds == 0 ? 3 : 0, step = gx >> xs, part = bx & ((1 << xs) - 1);   // (8 XCDs; shifts: a division is 40 instructions)
  const int first = (int)((long)tiles * part >> xs) + (bx >> xs), end = (int)((long)tiles * (part + 1) >> xs);
  if (first >= end) return;

  // ---- the filter: [32 channels][step][lane] 16 bytes
  u32x4 w[9][KS];
  {
    const u32x4* const src = (const u32x4*)p.wd + (size_t)(co0 / 32) * p.k_steps * 64 + lane;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int k = 0; k < KS; ++k) w[t][k] = src[(t * KS + k) * 64];
  }

  // ---- the slots this lane fetches of every patch: byte offset from the patch's first pixel, row and column
  const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.x), 0, (int)((size_t)p.N * p.x_rows * p.W * PIXB), 0x00020000);
  unsigned rel[NI];
  int at_px[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int slot = (i * 4 + wave) * 64 + lane;
    const int pix = slot / SLOTS, k = slot - pix * SLOTS;
    const int pr = smalldiv(pix, p.by_pitch), pc = pix - pr * p.pitch, half_cols = p.pitch >> 1;
    const int col = S == 1 ? pc : (pc < half_cols ? 2 * pc : 2 * (pc - half_cols) + 1);
    const bool ok = (k < SLOTS - 1) & (pr < p.ph_rows);
    rel[i] = ok ? (unsigned)((pr * p.W + col) * PIXB + k * 16) : kOutside;
    at_px[i] = pr << 16 | col;
  }
  struct At { int n, r0, c0; };
  auto tile_at = [&](int t) __attribute__((always_inline)) {
    const int q = fastdiv(t, p.by_ntx), n = fastdiv(q, p.by_nty);
    return At{n, (q - n * p.nty) * p.th, (t - q * p.ntx) * p.tw};
  };
  auto fetch_patch = [&](const At& a, int buf) __attribute__((always_inline)) {
    const int ih0 = (p.out_lo + a.r0) * S - p.ph, iw0 = a.c0 * S - p.pw;
    const int base = ((a.n * p.x_rows + ih0 - p.x_row0) * p.W + iw0) * PIXB;
    const bool inside = ih0 >= p.x_row0 && ih0 + p.ph_rows <= p.x_row0 + p.x_rows && iw0 >= 0 && iw0 + p.pitch <= p.W;
    unsigned char* const dst = smem + buf * BUF;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      bool ok = rel[i] != kOutside;
      if (!inside) {   // a pixel outside the image or the slab is a load past the buffer's end
        const int ih = ih0 + (at_px[i] >> 16), iw = iw0 + (at_px[i] & 0xffff);
        ok = ok & (ih >= p.x_row0) & (ih < p.x_row0 + p.x_rows) & (iw >= 0) & (iw < p.W);
      }
      const int src = ok ? (int)rel[i] + base : (int)kOutside;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (__attribute__((address_space(3))) void*)(dst + (i * 4 + wave) * 1024), 16, src, 0, 0, 0);
    }
  };

  // ---- this lane's pixel of its wavefront's 32: row and column inside a tile, where it lies in a patch
  int pr, pc;
  {
    const int i = frag * 32 + px;
    if constexpr (POOL) {   // window by window, so that a window is four neighbouring lanes
      const int v = i >> 2, vr = smalldiv(v, p.by_tw), vc = v - vr * (p.tw >> 1);   // (by_tw divides by tw / 2)
      pr = vr * 2 + ((i >> 1) & 1);
      pc = vc * 2 + (i & 1);
    } else {
      pr = smalldiv(i, p.by_tw);
      pc = i - pr * p.tw;
    }
  }
  const bool stores = pr < p.th && (!POOL || (lane & 3) == 0);
  // (lanes past the tile compute its last row again; they store nothing)
  const int at = (int)(unsigned)(unsigned long)(__attribute__((address_space(3))) unsigned char*)smem +
                 ((min(pr, p.th - 1) * S) * p.pitch + pc) * PB + half * 16;
  const int tap_row = p.pitch * PB, tap_odd = (p.pitch >> 1) * PB;
  f32x4 bias[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) bias[g] = p.bias ? *(const f32x4*)(p.bias + co0 + g * 8 + half * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
  const Clamp cl = make_clamp(p.act);

  // a tile's results: two 16-byte pieces per lane, and where they go
  u32x4 out[2];
  size_t out_at = 0;
  bool out_live = false;
  auto store_out = [&]() __attribute__((always_inline)) {
    if (!out_live) return;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      *(u32x4*)((__bf16*)p.y + out_at + i * 16) = out[i];
      if (p.y2) *(u32x4*)((__bf16*)p.y2 + out_at + i * 16) = out[i];
    }
  };

  At a = tile_at(first);
  fetch_patch(a, 0);
  for (int t = first, buf = 0;; t += step, buf ^= 1) {
    // the patch has arrived, and every wavefront is done with the other buffer
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    store_out();
    const int row = a.r0 + pr, col = a.c0 + pc;
    out_live = stores & (row < p.R) & (col < p.Wc);
    uint2 res[4];
    if constexpr (!POOL) {
      out_at = ((size_t)(a.n * p.y_rows + p.out_lo + row - p.y_row0) * p.W_out + col) * p.C_out + co0 + half * 8;
      if (p.res) {   // (ahead of the next patch: a wait for these is then none for that)
        const size_t ra = out_live ? ((size_t)(a.n * p.r_rows + p.out_lo + row - p.r_row0) * p.W_out + col) * p.C_out + co0 : 0;
#pragma unroll
        for (int g = 0; g < 4; ++g) res[g] = *(const uint2*)((const __bf16*)p.res + ra + g * 8 + half * 4);
      }
      asm volatile("" ::: "memory");
    } else {
      out_at = ((size_t)(a.n * p.y_rows + ((p.out_lo + row) >> 1) - p.y_row0) * p.W_out + (col >> 1)) * p.C_out + co0 + half * 8;
    }
    const bool more = t + step < end;
    if (more) {
      a = tile_at(t + step);
      fetch_patch(a, buf ^ 1);
    }
    __builtin_amdgcn_sched_barrier(0);

    f32x16 acc;   // (starts from the bias; with pooling that is added behind the products, see max_of_quad)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = POOL ? 0.f : bias[i / 4][i % 4];
    const int here = at + buf * BUF;
    u32x4 x[AHEAD + 1][KS];   // a tap's pixels are read AHEAD taps before they are multiplied
    unroll<AHEAD>([&](auto tap) __attribute__((always_inline)) {
      constexpr int T = decltype(tap)::value;
      read_tap<S, PB, KS, T>(here, tap_row, tap_odd, x[T]);
    });
    unroll<9>([&](auto tap) __attribute__((always_inline)) {
      constexpr int T = decltype(tap)::value;
      if constexpr (T + AHEAD < 9) read_tap<S, PB, KS, T + AHEAD>(here, tap_row, tap_odd, x[(T + AHEAD) % (AHEAD + 1)]);
      wait_reads<(T + AHEAD < 9 ? AHEAD : 8 - T) * KS>(x[T % (AHEAD + 1)]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < KS; ++k) mma<__bf16>(w[T][k], x[T % (AHEAD + 1)][k], acc);
      __builtin_amdgcn_sched_barrier(0);
    });

    // ---- residual, pooling, activation, the one rounding; channels 8 g + 4 half + {0..3} become
    // 8 consecutive ones per lane by an exchange between the lane halves
    if constexpr (!POOL) {
      if (p.res) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          alignas(8) __bf16 rr[4];
          *(uint2*)rr = res[g];
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[g * 4 + j] += (float)rr[j];
        }
      }
    }
    uint2 o[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 v = f32x4{acc[g * 4], acc[g * 4 + 1], acc[g * 4 + 2], acc[g * 4 + 3]};
      if constexpr (POOL) {
        max_of_quad(v, bias[g]);
      }
      alignas(8) __bf16 b[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = (__bf16)clamp_act(v[j], cl);
      o[g] = *(const uint2*)b;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const auto s0 = __builtin_amdgcn_permlane32_swap(o[2 * i].x, o[2 * i + 1].x, false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(o[2 * i].y, o[2 * i + 1].y, false, false);
      out[i] = u32x4{(unsigned)s0[0], (unsigned)s1[0], (unsigned)s0[1], (unsigned)s1[1]};
    }
    if (!more) break;
  }
  store_out();
}

template <int PIXB, int S, int WCO, bool POOL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PIXB == 64 ? 3 : 2))) void conv_walk_kernel(const PatchParams p) {
  walk_body<PIXB, S, WCO, POOL>(p, blockIdx.x, gridDim.x);
}
// The same for several bands of one layer in one grid (band b owns blocks first[b] .. first[b + 1] of x).
template <int PIXB, int S, int WCO, bool POOL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PIXB == 64 ? 3 : 2))) void conv_walk_kernel_bands(const Batch<PatchParams> t) {
  const int b = batch_find(t, blockIdx.x);
  walk_body<PIXB, S, WCO, POOL>(t.p[b], blockIdx.x - t.first[b], t.first[b + 1] - t.first[b]);
}

// The form of a launch: pixels of 64 or 128 bytes, stride, blocks of channels per workgroup (0: none), the
// workgroups that are resident at once.
struct WalkForm { int pixb, s, wco, pixels, room; long resident; };
template <int PIXB, int S, int WCO>
constexpr WalkForm walk_form() {
  return {PIXB, S, WCO, WalkTile<PIXB, S, WCO>::PIXELS, WalkTile<PIXB, S, WCO>::ROOM, PIXB == 64 ? 768 : 512};
}

long walk_pixels(const OpLaunch* convs, const OpLaunch* pools, int n) {
  long m = 0;
  for (int b = 0; b < n; ++b) {
    const PatchWork w = patch_work(convs[b], pools ? &pools[b] : nullptr);
    if (w.R > 0) m += (long)w.N * w.R * w.Wc;
  }
  return m;
}

// Whether a launch is large enough, in output elements (of the convolution itself): below, the tiles do not go round the
// resident workgroups often enough to pay for loading the filter, and the kernels with one tile per
// workgroup are level or faster. Measured against them (us a launch; before -> here):
//   32 -> 32 channels on 856 000 pixels 36.5 -> 26, on 57 600 8.3 -> 5.6, on 32 400 5.6 -> 5.7;
//   64 -> 64 on 203 000 pixels 33 -> 25, pooled on 251 000 35.6 -> 26.8, on 57 600 10.3 -> 9.5, on 28 800 6.5 -> 7.0;
//   stride 2: 32 -> 64 on 106 000 pixels 40 -> 18.5, on 57 600 12.2 -> 7.7, on 14 400 5.3 -> 4.9, on 8 160 4.4 -> 5.1;
//   64 -> 128 on 49 600 22.7 -> 16.4, on 7 200 6.1 -> 5.3.
// What bounds the large ones now: instructions. A wavefront has 340 of them a tile (120 vector, 130 scalar, 18 or 36 of
// each of matrix products and reads from LDS) and issues one in four cycles at best; leaving out any one kind of memory access
// or the products changes 5 to 20 %. The bias as the sum's start, the residual's additions only where there is one
// and pooling in two instructions a value: 23.3 -> 22.0 us for 32 -> 32 on 857 000 pixels, 25.7 -> 24.9 pooled on 256 000.
constexpr long kMinOutputsStride2 = 900000, kMinOutputs32 = 1500000, kMinOutputs64 = 2750000;

WalkForm choose_walk(const OpLaunch* convs, const OpLaunch* pools, int n) {
  const WalkForm none = {0, 0, 0, 0, 0, 0};
  const OpLaunch& L = convs[0];
  if (L.op != LOP_CONV2D || L.dtype != LOP_BF16 || !L.wd || L.kh != 3 || L.kw != 3 || L.dh != 1 || L.dw != 1 || L.sh != L.sw) return none;
  for (int b = 0; b < n; ++b)   // 32-bit signed byte offsets into the input slab
    if ((size_t)convs[b].x.n * convs[b].x.rows * convs[b].x.w * convs[b].x.c * 2 >= ((size_t)1 << 31)) return none;
  const int c = L.x.c;
  const long outputs = walk_pixels(convs, pools, n) * L.y.c;
  if (outputs < (L.sh == 2 ? kMinOutputsStride2 : c == 32 ? kMinOutputs32 : kMinOutputs64)) return none;
  if (c == 32 && L.sh == 1 && L.y.c % 32 == 0 && !pools) return walk_form<64, 1, 1>();
  if (c == 32 && L.sh == 2 && L.y.c % 64 == 0 && !pools) return walk_form<64, 2, 2>();
  if (c == 64 && L.sh == 1 && L.y.c % 64 == 0) return walk_form<128, 1, 2>();
  if (c == 64 && L.sh == 2 && L.y.c % 128 == 0 && !pools) return walk_form<128, 2, 4>();
  return none;
}

}  // namespace

bool walk_applies(const OpLaunch* convs, const OpLaunch* pools, int n) {
  return n >= 1 && n <= kMaxBatch && choose_walk(convs, pools, n).pixb != 0;
}

hipError_t launch_walk(const OpLaunch* convs, const OpLaunch* pools, int n, hipStream_t s, KernelEvents* ev) {
  if (n < 1 || n > kMaxBatch) return hipErrorInvalidValue;
  const WalkForm f = choose_walk(convs, pools, n);
  if (!f.pixb) return hipErrorInvalidValue;
  const unsigned gy = (unsigned)(convs[0].y.c / (32 * f.wco));
  PatchParams ps[kMaxBatch];
  unsigned gx[kMaxBatch];
  int m = 0;
  long all = 0;
  for (int b = 0; b < n; ++b) {
    if (patch_work(convs[b], pools ? &pools[b] : nullptr).R <= 0) continue;
    ps[m] = make_patch(convs[b], pools ? &pools[b] : nullptr, f.pixels, f.room, gy, &gx[m]);
    const PatchParams& p = ps[m];
    if (p.th < 1 || p.th * p.tw > f.pixels || p.ph_rows * p.pitch > f.room || p.C_in * 2 != f.pixb) return hipErrorInvalidValue;
    all += gx[m++];
  }
  if (m == 0) return hipSuccess;
  // every band gets its share of the resident workgroups (a multiple of the XCD count), or one per
  // tile where those are fewer
  for (int b = 0; b < m; ++b) {
    const long tiles = gx[b], share = f.resident / gy * tiles / all / kXcds * kXcds;
    gx[b] = (unsigned)(share >= kXcds && share < tiles ? share : tiles);
  }
  const dim3 block(256);
  if (f.pixb == 64 && f.s == 1)
    return launch_group(conv_walk_kernel<64, 1, 1, false>, conv_walk_kernel_bands<64, 1, 1, false>, ps, m, gx, gy, 1, block, s, ev);
  if (f.pixb == 64)
    return launch_group(conv_walk_kernel<64, 2, 2, false>, conv_walk_kernel_bands<64, 2, 2, false>, ps, m, gx, gy, 1, block, s, ev);
  if (f.s == 2)
    return launch_group(conv_walk_kernel<128, 2, 4, false>, conv_walk_kernel_bands<128, 2, 4, false>, ps, m, gx, gy, 1, block, s, ev);
  if (pools)
    return launch_group(conv_walk_kernel<128, 1, 2, true>, conv_walk_kernel_bands<128, 1, 2, true>, ps, m, gx, gy, 1, block, s, ev);
  return launch_group(conv_walk_kernel<128, 1, 2, false>, conv_walk_kernel_bands<128, 1, 2, false>, ps, m, gx, gy, 1, block, s, ev);
}

int walk_describe(const OpLaunch* convs, const OpLaunch* pools, int n, char* name, size_t size) {
  const WalkForm f = choose_walk(convs, pools, n);
  int m = 0;
  for (int b = 0; b < n; ++b) m += patch_work(convs[b], pools ? &pools[b] : nullptr).R > 0;
  const char* const form = m > 1 ? "_bands" : "";
  if (name && size) snprintf(name, size, "conv_walk_kernel%s<%d, %d, %d, %s>", form, f.pixb, f.s, f.wco, pools ? "true" : "false");
  return 1;
}

}  // namespace lop
