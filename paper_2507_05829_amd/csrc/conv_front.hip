// A 3 x 3 first layer over RGB images and the 3 x 3 stride-1 convolution of its 32 or 64 channels behind it (bf16; with or
// without the 2 x 2 max pooling behind that) as one launch.
//
// As two, the first layer is bound by the output that it writes, and the second one reads it back: at 720p with 16 bands 54 MB
// each way. Here a workgroup walks over tiles of the second layer's output with both filters in registers, like the walking
// kernel (conv_walk.hip). For a tile it stages the image rows under it in LDS (4 bytes per load, on their way while the tile before is
// worked on), computes the first layer's pixels under the tile's windows (1.3 to 1.4 times the tile's: halos are computed again) into a
// patch in LDS, zero where they lie outside that layer's image (the second layer's padding), and multiplies 64 pixels by 32
// channels per wavefront over the whole reduction. Products, sums and roundings are those of the first layer's own launch and of
// the walking kernel, in their order: the bits are the same wherever those two are what it stands for.
// What bounds it: a tile's chain of image, first layer, second layer between two barriers, with two or three workgroups on a
// compute unit. Bounds, masks and zeros only at the borders. (The first layer's sums started from its bias would save 16
// additions for 32 of its pixels and no time that can be measured, 136.3 and 136.6 us, but are not that layer's bits.)
// (What it is worth, measured: see kFrontTiles64.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "act.hpp"
#include "conv_common.hpp"
#include "conv_tiles.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

struct FrontParams {
  const void* x;
  void* y;
  void* y2;            // second destination with y's layout, or nullptr
  const void* w1;      // first layer: [C / 32][filter row][lane] 16 bytes
  const void* w2;      // second layer: [32 channels][step][lane] 16 bytes
  const float* b1;
  const float* b2;
  int x_row0, x_rows, W;               // image rows in the slab, its width
  int ph1, pw1, act1, H1, W1;          // first layer; its output's size
  int y_row0, y_rows, W_out;           // of the tensor that is stored
  int ph, pw, act, k_steps, C_out, out_lo, R, N, Wc;
  int th, tw, nty, ntx, pitch, ph_rows;   // tile of output pixels; pixels per row of the patch, its rows
  int img_rows, img_words;                // image rows under a patch, 4-byte words of one (odd: rows start on different banks)
  FastDiv by_ntx, by_nty, by_words, by_rows;
  unsigned by_tw, by_pitch;          // (small_div)
};
static_assert(sizeof(Batch<FrontParams>) <= 4096, "the parameters of all bands of a launch travel as kernel arguments");

// S1: stride of the first layer; NT: blocks of 32 channels
template <int S1, int NT>
struct FrontTile {
  static constexpr int PB = NT * 64 + 16;                 // bytes of a pixel of the patch: an odd number of 16-byte slots
  static constexpr int KS = NT * 2;                       // reduction steps of a tap
  static constexpr int PIXELS = 256 / NT;                 // two fragments of 32 a wavefront
  static constexpr int ROOM = NT == 1 ? 352 : 192;        // pixels of a patch
  static constexpr int MID = (ROOM / 32 + 3) / 4;         // its fragments per wavefront
  static constexpr int COPIES = S1 == 1 ? 2 : 1;          // of the image rows: with stride 1 every second window starts between two words
  static constexpr int LOADS = NT == 1 ? (S1 == 1 ? 6 : 9) : (S1 == 1 ? 4 : 6);   // words of them per thread
  static constexpr int WORDS = LOADS * 256;
};

template <int S1, int NT, bool POOL>
__device__ __forceinline__ void front_body(const FrontParams& p, const int bx, const int gx) {
  typedef FrontTile<S1, NT> G;
  constexpr int PB = G::PB, KS = G::KS, MID = G::MID, COPIES = G::COPIES, LOADS = G::LOADS;
  __shared__ __attribute__((aligned(16))) unsigned char patch_s[G::ROOM * PB];
  __shared__ __attribute__((aligned(16))) float bias_s[2][NT * 32];
  __shared__ unsigned image_s[G::WORDS + 16];             // (the last windows' groups end behind the last row)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int px = lane & 31, half = lane >> 5;
  const int co0 = (NT == 1 ? 0 : wave & 1) * 32, group = NT == 1 ? wave : wave >> 1;   // channels and 64 pixels of this wavefront

  // ---- this workgroup's tiles: first, first + step, ... below end (XCD k walks the k-th eighth)
  const int tiles = p.N * p.nty * p.ntx;
  const int xs = (unsigned)gx % kXcds == 0 ? 3 : 0, step = gx >> xs, part = bx & ((1 << xs) - 1);   // (8 XCDs)
  const int first = (int)((long)tiles * part >> xs) + (bx >> xs), end = (int)((long)tiles * (part + 1) >> xs);
  if (first >= end) return;

  // ---- the words this thread stages of every tile, [copy][row][word]: the i-th is i * 256 + tid (the last one again
  // past it, into memory nobody reads). Row and element of it:
  const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(p.x), 0, (int)((size_t)p.N * p.x_rows * p.W * 6), 0x00020000);
  auto word_at = [&](int word, int& r, int& e) __attribute__((always_inline)) {
    const int idx = min(word, p.img_rows * p.img_words * COPIES - 1);
    const int cr = fastdiv(idx, p.by_words), c = COPIES == 1 ? 0 : fastdiv(cr, p.by_rows);
    r = cr - c * p.img_rows;
    e = (idx - cr * p.img_words) * 2 + c;
  };
  unsigned rel[LOADS];          // element offset from the tile's first image element
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    int r, e;
    word_at(i * 256 + tid, r, e);
    rel[i] = (unsigned)(r * p.W * 3 + e);
  }
  struct At { int n, r0, c0; };
  auto tile_at = [&](int t) __attribute__((always_inline)) {
    const int q = fastdiv(t, p.by_ntx), n = fastdiv(q, p.by_nty);
    return At{n, (q - n * p.nty) * p.th, (t - q * p.ntx) * p.tw};
  };
  unsigned raw[LOADS];
  auto fetch = [&](const At& a) __attribute__((always_inline)) {
    const int ih0 = (p.out_lo + a.r0 - p.ph) * S1 - p.ph1, e0 = ((a.c0 - p.pw) * S1 - p.pw1) * 3, row_elems = p.W * 3;
    const unsigned short* const base = (const unsigned short*)p.x + ((long)(a.n * p.x_rows + ih0 - p.x_row0) * row_elems + e0);
    const bool inside = ih0 >= p.x_row0 && ih0 + p.img_rows <= p.x_row0 + p.x_rows && e0 >= 0 && e0 + 2 * p.img_words + COPIES - 1 <= row_elems;
    if (inside) {
#pragma unroll
      for (int i = 0; i < LOADS; ++i) __builtin_memcpy(&raw[i], base + rel[i], 4);
    } else {   // two halves of a word, each zero outside the image and the slab (a load past the buffer's end)
      int t = tid;
      asm volatile("" : "+v"(t));   // (worked out anew: kept over the tiles, rows and elements would not fit the registers)
#pragma unroll
      for (int i = 0; i < LOADS; ++i) {
        int r, e;
        word_at(i * 256 + t, r, e);
        const int ih = ih0 + r;
        e += e0;
        const bool row_ok = ih >= p.x_row0 && ih < p.x_row0 + p.x_rows;
        const int at = ((a.n * p.x_rows + ih - p.x_row0) * row_elems + e) * 2;
        const unsigned lo = __builtin_amdgcn_raw_buffer_load_b16(xbuf, row_ok & (e >= 0) & (e < row_elems) ? at : (int)kOutside, 0, 0);
        const unsigned hi = __builtin_amdgcn_raw_buffer_load_b16(xbuf, row_ok & (e + 1 >= 0) & (e + 1 < row_elems) ? at + 2 : (int)kOutside, 0, 0);
        raw[i] = lo | hi << 16;
      }
    }
  };

  At a = tile_at(first);
  fetch(a);
  // ---- the filters
  u32x4 w1[3][NT], w2[9][KS];
#pragma unroll
  for (int k = 0; k < NT; ++k)
#pragma unroll
    for (int t = 0; t < 3; ++t) w1[t][k] = ((const u32x4*)p.w1)[(k * 3 + t) * 64 + lane];
  {
    const u32x4* const src = (const u32x4*)p.w2 + (size_t)(co0 / 32) * p.k_steps * 64 + lane;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int k = 0; k < KS; ++k) w2[t][k] = src[(t * KS + k) * 64];
  }
  if (tid < NT * 32) {
    bias_s[0][tid] = p.b1 ? p.b1[tid] : 0.f;
    bias_s[1][tid] = p.b2 ? p.b2[tid] : 0.f;
  }
  const Clamp cl1 = make_clamp(p.act1), cl = make_clamp(p.act);

  // ---- this lane's pixels of the patch: where their windows start in the staged image
  const int count = p.ph_rows * p.pitch;
  auto middle_pixel = [&](int m) { return min((wave + 4 * m) * 32 + px, count - 1); };
  int win[MID];
#pragma unroll
  for (int m = 0; m < MID; ++m) {
    const int i = middle_pixel(m), r = smalldiv(i, p.by_pitch), c = i - r * p.pitch;
    const int e = c * S1 * 3;
    win[m] = ((COPIES == 2 ? (e & 1) * p.img_rows : 0) + r * S1) * p.img_words + e / 2 + half * 4;
  }
  // ... and of the tile: row and column (16 bits each), where the first tap lies in the patch
  int rc[2], at[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int i = (group * 2 + f) * 32 + px;
    int r, c;
    if constexpr (POOL) {   // window by window, so that a window is four neighbouring lanes
      const int v = i >> 2, vr = smalldiv(v, p.by_tw), vc = v - vr * (p.tw >> 1);   // (by_tw divides by tw / 2)
      r = vr * 2 + ((i >> 1) & 1);
      c = vc * 2 + (i & 1);
    } else {
      r = smalldiv(i, p.by_tw);
      c = i - r * p.tw;
    }
    rc[f] = r << 16 | c;
    // (lanes past the tile compute its last row again; they store nothing)
    at[f] = (min(r, p.th - 1) * p.pitch + c) * PB + half * 16;
  }
  auto barrier = [&]() __attribute__((always_inline)) {   // (for LDS only: loads and stores stay in flight)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  for (int t = first;; t += step) {
    // ---- the image under the tile (nobody reads the one before it any more)
#pragma unroll
    for (int i = 0; i < LOADS; ++i) image_s[i * 256 + tid] = raw[i];
    barrier();
    const At now = a;
    const bool more = t + step < end;
    if (more) {
      a = tile_at(t + step);
      fetch(a);
    }
    // ---- the first layer's pixels under the tile's windows
    const unsigned upper = half ? 0u : 0xffffffffu;
    const int h_first = p.out_lo + now.r0 - p.ph, c_first = now.c0 - p.pw;   // of the patch, in that layer's image
    auto middle = [&](auto masked) __attribute__((always_inline)) {
#pragma unroll
      for (int m = 0; m < MID; ++m) {
        if ((wave + 4 * m) * 32 >= count) continue;
        f32x16 acc[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[k][i] = 0.f;
#pragma unroll
        for (int r = 0; r < 3; ++r) {   // a filter row: elements 0 .. 7 in the lower half of the wavefront, element 8 in the upper
          const unsigned* const src = image_s + win[m] + r * p.img_words;
          const u32x4 d = u32x4{src[0] & (upper | 0xffffu), src[1] & upper, src[2] & upper, src[3] & upper};
#pragma unroll
          for (int k = 0; k < NT; ++k) mma<__bf16>(w1[r][k], d, acc[k]);
        }
        int i = middle_pixel(m);
        unsigned char* const to = patch_s + i * PB + half * 8;
        bool in = true;
        if constexpr (masked) {
          asm volatile("" : "+v"(i));   // (row and column worked out anew, like a border tile's words)
          const int r = smalldiv(i, p.by_pitch), c = i - r * p.pitch;
          in = (h_first + r >= 0) & (h_first + r < p.H1) & (c_first + c >= 0) & (c_first + c < p.W1);
        }
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
          for (int g = 0; g < 4; ++g) {   // (the bias behind the products, as the layer's own launch adds it)
            const f32x4 b = *(const f32x4*)(bias_s[0] + k * 32 + g * 8 + half * 4);
            alignas(8) __bf16 o[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = (__bf16)clamp_act(acc[k][g * 4 + j] + b[j], cl1);
            uint2 v = *(const uint2*)o;
            if (masked && !in) v = make_uint2(0u, 0u);
            *(uint2*)(to + k * 64 + g * 16) = v;
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (h_first >= 0 && h_first + p.ph_rows <= p.H1 && c_first >= 0 && c_first + p.pitch <= p.W1) middle(std::false_type{});
    else middle(std::true_type{});
    barrier();

    // ---- the second layer
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      f32x4 bias[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) bias[g] = *(const f32x4*)(bias_s[1] + co0 + g * 8 + half * 4);
      f32x16 acc;   // (starts from the bias; with pooling that is added behind the products, see max_of_quad)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = POOL ? 0.f : bias[i / 4][i % 4];
      const unsigned char* const here = patch_s + at[f];
      u32x4 x[2][KS];   // a tap's pixels are read while the one before is multiplied
      auto read = [&](int tap, u32x4 (&d)[KS]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < KS; ++k) d[k] = *(const u32x4*)(here + (tap / 3 * p.pitch + tap % 3) * PB + k * 32);
      };
      read(0, x[0]);
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        if (tap < 8) read(tap + 1, x[(tap + 1) & 1]);
#pragma unroll
        for (int k = 0; k < KS; ++k) mma<__bf16>(w2[tap][k], x[tap & 1][k], acc);
        __builtin_amdgcn_sched_barrier(0);
      }
      uint2 o[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 v = f32x4{acc[g * 4], acc[g * 4 + 1], acc[g * 4 + 2], acc[g * 4 + 3]};
        if constexpr (POOL) max_of_quad(v, bias[g]);
        alignas(8) __bf16 b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = (__bf16)clamp_act(v[j], cl);
        o[g] = *(const uint2*)b;
      }
      const int row = now.r0 + (rc[f] >> 16), col = now.c0 + (rc[f] & 0xffff);
      const bool live = (rc[f] >> 16 < p.th) & (row < p.R) & (col < p.Wc) & (!POOL || (lane & 3) == 0);
      size_t ya;
      if constexpr (POOL) ya = ((size_t)(now.n * p.y_rows + ((p.out_lo + row) >> 1) - p.y_row0) * p.W_out + (col >> 1)) * p.C_out + co0 + half * 8;
      else ya = ((size_t)(now.n * p.y_rows + p.out_lo + row - p.y_row0) * p.W_out + col) * p.C_out + co0 + half * 8;
#pragma unroll
      for (int i = 0; i < 2; ++i) {   // channels 8 g + 4 half + {0..3} become 8 consecutive ones per lane
        const auto s0 = __builtin_amdgcn_permlane32_swap(o[2 * i].x, o[2 * i + 1].x, false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(o[2 * i].y, o[2 * i + 1].y, false, false);
        const u32x4 v = u32x4{(unsigned)s0[0], (unsigned)s1[0], (unsigned)s0[1], (unsigned)s1[1]};
        if (live) {
          *(u32x4*)((__bf16*)p.y + ya + i * 16) = v;
          if (p.y2) *(u32x4*)((__bf16*)p.y2 + ya + i * 16) = v;
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // (one fragment's reads at a time: registers)
    }
    if (!more) return;
  }
}

template <int S1, int NT, bool POOL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NT == 1 ? 3 : 2))) void conv_front_kernel(const FrontParams p) {
  front_body<S1, NT, POOL>(p, blockIdx.x, gridDim.x);
}
// The same for several bands in one grid (band b owns blocks first[b] .. first[b + 1]).
template <int S1, int NT, bool POOL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NT == 1 ? 3 : 2))) void conv_front_kernel_bands(const Batch<FrontParams> t) {
  const int b = batch_find(t, blockIdx.x);
  front_body<S1, NT, POOL>(t.p[b], blockIdx.x - t.first[b], t.first[b + 1] - t.first[b]);
}

struct FrontForm { int s1 = 0, nt = 0, pixels = 0, room = 0, words = 0, copies = 0; };
template <int S1, int NT>
constexpr FrontForm front_form() {
  typedef FrontTile<S1, NT> G;
  return FrontForm{S1, NT, G::PIXELS, G::ROOM, G::WORDS, G::COPIES};
}

// Parameters of a band; false where a tile does not fit.
bool make_front(const OpLaunch& a, const OpLaunch& c, const OpLaunch* pool, const FrontForm& f, FrontParams* out, unsigned* tiles) {
  unsigned n = 0;
  const PatchParams q = make_patch(c, pool, f.pixels, f.room, 1, &n);
  FrontParams p;
  p.x = a.x.ptr; p.y = q.y; p.y2 = q.y2;
  p.w1 = (const char*)a.wstem + stem_mfma_offset(a.x.c, a.y.c, a.kh, a.kw); p.w2 = c.wd; p.b1 = a.bias; p.b2 = c.bias;
  p.x_row0 = a.x.row0; p.x_rows = a.x.rows; p.W = a.x.w;
  p.ph1 = a.ph; p.pw1 = a.pw; p.act1 = a.act; p.H1 = c.x.h; p.W1 = c.x.w;
  p.y_row0 = q.y_row0; p.y_rows = q.y_rows; p.W_out = q.W_out;
  p.ph = q.ph; p.pw = q.pw; p.act = q.act; p.k_steps = q.k_steps; p.C_out = q.C_out; p.out_lo = q.out_lo; p.R = q.R; p.N = q.N; p.Wc = q.Wc;
  p.th = q.th; p.tw = q.tw; p.nty = q.nty; p.ntx = q.ntx; p.pitch = q.pitch; p.ph_rows = q.ph_rows;
  // windows of 3 rows x 16 elements (9 of them live) at S1 x 3 elements from each other
  p.img_rows = (q.ph_rows - 1) * f.s1 + 3;
  p.img_words = ((q.pitch - 1) * f.s1 * 3 + 9 + 1) / 2 | 1;
  p.by_ntx = q.by_ntx; p.by_nty = q.by_nty; p.by_tw = q.by_tw; p.by_pitch = q.by_pitch;
  p.by_words = make_fastdiv(p.img_words); p.by_rows = make_fastdiv(p.img_rows);
  *out = p;
  *tiles = n;
  return q.th >= 1 && q.th * q.tw <= f.pixels && q.ph_rows * q.pitch <= f.room && p.img_rows * p.img_words * f.copies <= f.words;
}

FrontForm choose_front(const OpLaunch& a, const OpLaunch& c, const OpLaunch* pool) {
  if (a.op != LOP_CONV2D || c.op != LOP_CONV2D || a.dtype != LOP_BF16 || c.dtype != LOP_BF16 || !a.wstem || !c.wd) return {};
  if (a.kh != 3 || a.kw != 3 || a.dh != 1 || a.dw != 1 || !stem_applies(a) || !stem_mfma_applies(a) || a.res.ptr || c.res.ptr) return {};
  if (c.kh != 3 || c.kw != 3 || c.sh != 1 || c.sw != 1 || c.dh != 1 || c.dw != 1 || c.x.c != a.y.c || c.y.c != a.y.c) return {};
  if (pool && (pool->kh != 2 || pool->kw != 2 || pool->sh != 2 || pool->sw != 2 || pool->ph != 0 || pool->pw != 0)) return {};
  if (a.y.c == 32 && !pool) return a.sh == 1 ? front_form<1, 1>() : front_form<2, 1>();
  if (a.y.c == 64) return a.sh == 1 ? front_form<1, 2>() : front_form<2, 2>();
  return {};
}

// With 64 channels: tiles a launch has at least. us a call with calls in flight and alone, two launches -> this one: detector
// encoder 720 x 1280 in 16 independent bands 146.2 -> 140.4, 289 -> 272, with shared rows 63.5 -> 61.7, 151 -> 141 (without the copy 51.7 -> 48.0, 111 ->
// 103), 250 x 333 in five bands 27.0 -> 24.5, 84 -> 81; 224 x 224 into 64 channels, eight independent bands 143.0 -> 139.0, 224 -> 218, with shared rows
// 43.5 -> 42.4, 110 -> 105; 128 x 128 27.9 -> 27.1, 83.5 -> 83.1; 96 x 96 (72 tiles) 26.7 -> 26.1, 82.5 -> 82.7; but 64 x 64 (32 tiles)
// 25.9 -> 25.6, 89.7 -> 91.2: a few workgroups then do one after the other what many do at once.
constexpr long kFrontTiles64 = 64;

size_t slab_bytes(const Slab& s) { return (size_t)s.n * s.rows * s.w * s.c * 2; }

}  // namespace

// pools: the 2 x 2 max pooling behind each band's second layer, or nullptr. (Whether the launch applies is found out while its parameters
// are made: with many small bands those are what a call costs.)
hipError_t launch_front(const OpLaunch* firsts, const OpLaunch* seconds, const OpLaunch* pools, int n, hipStream_t s, bool* taken,
                        KernelEvents* ev) {
  *taken = false;
  if (n < 1 || n > kMaxBatch) return hipSuccess;
  FrontForm f;
  FrontParams ps[kMaxBatch];
  unsigned gx[kMaxBatch];
  int m = 0;
  long all = 0;
  for (int b = 0; b < n; ++b) {
    const OpLaunch* const pool = pools ? &pools[b] : nullptr;
    f = choose_front(firsts[b], seconds[b], pool);
    const size_t x_bytes = slab_bytes(firsts[b].x);
    if (!f.nt || x_bytes >= ((size_t)1 << 31)) return hipSuccess;   // 32-bit offsets into the image
    // a workgroup stores its outputs while others still read the image
    const char* const x = (const char*)firsts[b].x.ptr;
    for (int j = 0; j < n; ++j) {
      const Slab& ys = pools ? pools[j].y : seconds[j].y;
      const char* const y = (const char*)ys.ptr;
      if (x < y + slab_bytes(ys) && y < x + x_bytes) return hipSuccess;
    }
    if (patch_work(seconds[b], pool).R <= 0) continue;
    if (!make_front(firsts[b], seconds[b], pool, f, &ps[m], &gx[m])) return hipSuccess;
    all += gx[m++];
  }
  if (f.nt == 2 && all < kFrontTiles64) return hipSuccess;
  *taken = true;
  if (m == 0) return hipSuccess;
  // every band gets its share of the resident workgroups (a multiple of the XCD count), or one per
  // tile where those are fewer
  const long resident = f.nt == 1 ? 768 : 512;
  for (int b = 0; b < m; ++b) {
    const long tiles = gx[b], share = resident * tiles / all / kXcds * kXcds;
    gx[b] = (unsigned)(share >= kXcds && share < tiles ? share : tiles);
  }
  const dim3 block(256);
#define LOP_FRONT(S1, NT, POOL) return launch_group(conv_front_kernel<S1, NT, POOL>, conv_front_kernel_bands<S1, NT, POOL>, ps, m, gx, 1, 1, block, s, ev)
  if (f.nt == 1) {
    if (f.s1 == 1) LOP_FRONT(1, 1, false);
    LOP_FRONT(2, 1, false);
  }
  if (f.s1 == 1) {
    if (pools) LOP_FRONT(1, 2, true);
    LOP_FRONT(1, 2, false);
  }
  if (pools) LOP_FRONT(2, 2, true);
  LOP_FRONT(2, 2, false);
#undef LOP_FRONT
}

}  // namespace lop
