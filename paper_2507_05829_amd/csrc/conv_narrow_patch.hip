// Dense 3 x 3 convolution of few pixels in fp32, the 16 x 16-tile kernel in its patch form.
//
// The last stages of a backbone have too few output pixels for the chip: 196 pixels x 256 channels are 56
// tiles of 32 x 32, and a tile's reduction (2 304 elements) takes four wavefronts 4 us of matrix
// instructions alone. A workgroup here owns 16 pixels x 16 channels (208 of them) and sixteen
// wavefronts that split the reduction. All it needs is in flight at once: the input pixels under its
// rectangle with all their channels (a "patch", at most kMaxPatch bytes: global -> LDS, contiguous
// pieces) and every wavefront's first kAhead filter vectors (registers, in operand order). So there
// is one round of memory latency, one barrier, the matrix instructions and the sum of the sixteen
// partial tiles through LDS. At most 64 registers, so that two workgroups share a compute unit (of the same
// launch or of another chain): 20.4 -> 17.4 us for 320 tiles of 512 -> 512 channels. What is left is the
// launch, that round of latency and, with 4 608 reduction elements, 4.4 us of matrix instructions.
//
// conv_narrow_patch_kernel of conv_igemm.hip, which this form replaces where the patch fits, gathers every
// tap of every pixel straight into operand registers: four lanes of such a load touch four cache lines, which
// costs the vector cache four times the cycles of a contiguous one, nine times over.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>

#include "act.hpp"
#include "conv_common.hpp"
#include "conv_tiles.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

struct NarrowParams {
  const float* x;
  float* y;
  float* y2;         // second destination with y's layout, or nullptr
  const float* res;
  const void* wd16;  // weights in the operand order of 16 x 16 tiles
  const float* bias;
  int x_row0, x_rows, W, C_in;
  int y_row0, y_rows, W_out, C_out;
  int r_row0, r_rows;
  int s, ph, pw, act, w_steps;       // w_steps: MFMA steps of a packed weight row
  int out_lo, R, N;
  int th, tw, nty, ntx;              // tile of output pixels, tiles per image in either direction
  int pitch, ph_rows;                // pixels per row of the patch, its rows
  // a 1 x 1 convolution of the same input and stride, in the channel tiles from b_first on (see Sibling)
  const void* b_wd16;
  float* b_y;
  const float* b_bias;
  int b_w_steps, b_y_row0, b_y_rows, b_C_out, b_act, b_lo, b_hi, b_first;
  FastDiv by_ntx, by_nty, by_group, by_slots;
  unsigned by_tw, by_pitch;          // (small_div)
};
static_assert(sizeof(Batch<NarrowParams>) <= 4096, "the parameters of all bands of a launch travel as kernel arguments");

constexpr int kWaves = 16;
// LDS of a workgroup: most patches fit the small form, which leaves room for other workgroups on the compute unit
constexpr int kSmallPatch = 48 * 1024, kMaxPatch = 80 * 1024;
// Steps of 16 reduction elements. Fewer than four per wavefront are over before sixteen wavefronts have started
// (64 -> 128 channels, stride 2, on 784 pixels 6.1 us against 5.4); beyond the maximum the matrix
// instructions of one tile alone exceed 5 us.
constexpr int kMinSteps = 64, kMaxSteps = 288;
// Workgroups: up to one per compute unit the kernel beats the patch form with larger tiles and the
// gathering kernels (256 -> 256 channels on 196 pixels 6.9 us a launch of its own, 12.3 there; 256 -> 512, stride 2, on
// 49 pixels 6.9 against 11.8); with more, the larger tiles catch up where they apply (128 -> 128 on 784
// pixels 7.5 either way, and four chains in flight are faster with them). Where only a reduction cut
// across workgroups and its finish kernel would be left it wins up to four rounds (512 -> 512 on
// 49 pixels 9.8 us against 14.1, on 126 pixels 17.4 against 24.1).
constexpr long kTilesAlways = 256, kTilesOverCut = 1024;
constexpr int kPartPitch = 20;          // fp32 pitch of a staged partial tile

template <int AHEAD, int LDS>
__device__ __forceinline__ void narrow_body(const NarrowParams& p, const int bx, const int gx) {
  constexpr int LOADS = (LDS / 1024 + kWaves - 1) / kWaves;   // of a wavefront
  static_assert(LDS % 1024 == 0 && LDS >= kWaves * 16 * kPartPitch * 4, "whole loads; the partial tiles");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int px = lane & 15, kq = lane >> 4;
  const TileId tile = xcd_tile(bx, gx, gridDim.y, 1, p.by_group);
  const bool second = tile.n >= p.b_first;
  const int tile_n = second ? tile.n - p.b_first : tile.n, co0 = tile_n * 16;
  const int q = fastdiv(tile.m, p.by_ntx), tx = tile.m - q * p.ntx;
  const int n = fastdiv(q, p.by_nty), ty = q - n * p.nty;
  const int r0 = ty * p.th, c0 = tx * p.tw;
  const int row_bytes = p.C_in * 4, slots = p.C_in / 4 + 1;   // 16-byte slots of a pixel: an odd number, against bank conflicts
  const int total = p.pitch * p.ph_rows * slots;

  const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p.x), 0, (int)((size_t)p.N * p.x_rows * p.W * row_bytes), 0x00020000);
  const int ih0 = (p.out_lo + r0) * p.s - p.ph - p.x_row0, iw0 = c0 * p.s - p.pw, rows = min(p.x_rows, ih0 + p.ph_rows);   // in the slab
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int first = (i * kWaves + wave) * 64;
    if (first >= total) continue;
    const int slot = first + lane;
    const int pix = fastdiv(slot, p.by_slots), k = slot - pix * slots;
    const int pr = smalldiv(pix, p.by_pitch), pc = pix - (int)__umul24(pr, p.pitch);
    const int ih = ih0 + pr, iw = iw0 + pc;
    // (a pixel outside the image or the slab is a load past the buffer's end, which puts zeros into LDS; products of 24
    // bits: a slab has fewer pixels than that)
    const bool ok = (k < slots - 1) & (ih >= 0) & (ih < rows) & ((unsigned)iw < (unsigned)p.W);
    const unsigned to = __umul24(__umul24(n * p.x_rows + ih, p.W) + iw, row_bytes) + k * 16, src = ok ? to : kOutside;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (__attribute__((address_space(3))) void*)(smem + first * 16), 16, (int)src, 0, 0, 0);
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  // ---- this wavefront's slice of the reduction: steps s0 .. s1, its filter vectors AHEAD steps ahead
  const int tap_steps = p.C_in / 16, steps = second ? tap_steps : 9 * tap_steps, per_wave = (steps + kWaves - 1) / kWaves;
  const int s0 = min(steps, wave * per_wave), s1 = min(steps, s0 + per_wave);
  const u32x4* const wsrc = (const u32x4*)(second ? p.b_wd16 : p.wd16) + (size_t)tile_n * (second ? p.b_w_steps : p.w_steps) * 64 + lane;
  u32x4 w[AHEAD];
  auto fetch = [&](int s) __attribute__((always_inline)) { return wsrc[(size_t)min(s, steps - 1) * 64]; };
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) w[u] = fetch(s0 + u);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  int tap = s0 / tap_steps, ci = (s0 - tap * tap_steps) * 64;   // ci: bytes into the pixel
  if (second) tap = 4;
  int ta = min(tap / 3, 2), tb = tap - tap / 3 * 3;
  const int pixel_bytes = slots * 16;
  int at;
  {
    const int r = smalldiv(px, p.by_tw), c = px - r * p.tw;
    // (lanes past the tile compute its last row again; they store nothing)
    at = (min(r, p.th - 1) * p.s * p.pitch + c * p.s) * pixel_bytes + kq * 16;
  }
  // the patch is complete when this wavefront's part of it has arrived (only the filter loads are
  // younger) and the others have got here, too
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(AHEAD));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  auto read_step = [&]() __attribute__((always_inline)) {   // this lane's operand of the next step
    const u32x4 v = *(const u32x4*)(smem + at + (ta * p.pitch + tb) * pixel_bytes + ci);
    ci += 64;
    if (ci == row_bytes) {
      ci = 0;
      if (++tb == 3) { tb = 0; ta = min(ta + 1, 2); }   // (the step behind the last one is read, but not used)
    }
    return v;
  };
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 a = read_step();
  for (int sb = s0; sb < s1; sb += AHEAD) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      if (sb + u >= s1) continue;
      const u32x4 next = read_step();
      const f32x4 wf = __builtin_bit_cast(f32x4, w[u]), xf = __builtin_bit_cast(f32x4, a);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[e], xf[e], acc, 0, 0, 0);
      if (sb + AHEAD < s1) w[u] = fetch(sb + AHEAD + u);
      a = next;
    }
  }

  // ---- the sixteen partial tiles, added in wavefront order through LDS (over the patch): a lane holds
  // channels kq * 4 + {0..3} of pixel px
  // (what they are added to is loaded before the others' are there; what the launch has none of, from the beginning of the
  // filter, and not used)
  const int e_px = lane >> 2, co = co0 + (lane & 3) * 4;
  const int r = smalldiv(e_px, p.by_tw), col = c0 + e_px - r * p.tw, row = r0 + r;
  const int C_out = second ? p.b_C_out : p.C_out;
  bool live = (r < p.th) & (row < p.R) & (col < p.W_out) & (co < C_out);
  if (second) live = live & (p.out_lo + row >= p.b_lo) & (p.out_lo + row < p.b_hi);
  const float* const bias = second ? p.b_bias : p.bias;
  const bool has_res = p.res && !second;
  f32x4 bias_v, res_v;
  if (wave == 0) {
    bias_v = *(const f32x4*)((bias ? bias : (const float*)p.wd16) + (bias && live ? co : 0));
    res_v = *(const f32x4*)((has_res ? p.res : (const float*)p.wd16) +
                            (has_res && live ? ((size_t)(n * p.r_rows + p.out_lo + row - p.r_row0) * p.W_out + col) * p.C_out + co : 0));
  }
  __syncthreads();
  float* const part = (float*)smem;
  *(f32x4*)(part + wave * (16 * kPartPitch) + px * kPartPitch + kq * 4) = acc;
  __syncthreads();
  if (wave != 0 || !live) return;
  f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < kWaves; ++s) v += *(const f32x4*)(part + s * (16 * kPartPitch) + e_px * kPartPitch + (lane & 3) * 4);
  if (bias) v += bias_v;
  if (has_res) v += res_v;
  const Clamp cl = make_clamp(second ? p.b_act : p.act);
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = clamp_act(v[j], cl);
  const size_t ya = ((size_t)(n * (second ? p.b_y_rows : p.y_rows) + p.out_lo + row - (second ? p.b_y_row0 : p.y_row0)) * p.W_out + col) * C_out + co;
  *(f32x4*)((second ? p.b_y : p.y) + ya) = v;
  if (p.y2 && !second) *(f32x4*)(p.y2 + ya) = v;
}

template <typename T, int AHEAD, int LDS>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(8))) void conv_narrow_patch_kernel(const NarrowParams p) {
  narrow_body<AHEAD, LDS>(p, blockIdx.x, gridDim.x);
}
// The same for several bands of one layer in one grid (band b owns blocks first[b] .. first[b + 1] of x).
template <typename T, int AHEAD, int LDS>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(8))) void conv_narrow_patch_kernel_bands(const Batch<NarrowParams> t) {
  const int b = batch_find(t, blockIdx.x);
  narrow_body<AHEAD, LDS>(t.p[b], blockIdx.x - t.first[b], t.first[b + 1] - t.first[b]);
}

// The rectangle of at most 16 output pixels for R x W of them: the fewest tiles, then the smallest
// patch, as long as the patch fits.
struct NarrowTile { int th = 0, tw = 0; long tiles = 0; int patch = 0; };
NarrowTile narrow_tile(const OpLaunch& L) {
  const int R = L.out_hi - L.out_lo, W = L.y.w, s = L.sh, room = kMaxPatch / (L.x.c * 4 + 16);
  NarrowTile best;
  for (int tw = 1; tw <= std::min(16, W); ++tw) {
    int th = std::min(16 / tw, R);
    const int cols = (tw - 1) * s + 3;
    while (th >= 1 && ((th - 1) * s + 3) * cols > room) --th;
    if (th < 1) continue;
    const long tiles = (long)((R + th - 1) / th) * ((W + tw - 1) / tw) * L.x.n;
    const int patch = ((th - 1) * s + 3) * cols;
    if (!best.th || tiles < best.tiles || (tiles == best.tiles && patch < best.patch)) best = {th, tw, tiles, patch};
  }
  return best;
}

bool narrow_shape(const OpLaunch& L) {
  if (L.op != LOP_CONV2D || L.dtype == LOP_BF16 || !L.wd16 || L.kh != 3 || L.kw != 3 || L.dh != 1 || L.dw != 1) return false;
  if (L.sh != L.sw || (L.sh != 1 && L.sh != 2) || L.x.c % 16 != 0 || L.y.c % 4 != 0) return false;
  if (9 * L.x.c / 16 < kMinSteps || 9 * L.x.c / 16 > kMaxSteps) return false;
  return (size_t)L.x.n * L.x.rows * L.x.w * L.x.c * 4 < ((size_t)1 << 31);
}

long narrow_tiles(const OpLaunch* Ls, int n) {
  long t = 0;
  for (int b = 0; b < n; ++b) {
    if (Ls[b].out_hi <= Ls[b].out_lo) continue;
    const NarrowTile nt = narrow_tile(Ls[b]);
    if (!nt.th) return 0;
    t += nt.tiles;
  }
  return t * ((Ls[0].y.c + 15) / 16);
}

NarrowParams make_narrow(const OpLaunch& L, unsigned gy, unsigned* gx) {
  NarrowParams p;
  p.x = (const float*)L.x.ptr; p.y = (float*)L.y.ptr; p.y2 = (float*)L.y2; p.res = (const float*)L.res.ptr;
  p.wd16 = L.wd16; p.bias = L.bias;
  p.x_row0 = L.x.row0; p.x_rows = L.x.rows; p.W = L.x.w; p.C_in = L.x.c;
  p.y_row0 = L.y.row0; p.y_rows = L.y.rows; p.W_out = L.y.w; p.C_out = L.y.c;
  p.r_row0 = L.res.row0; p.r_rows = L.res.rows;
  p.s = L.sh; p.ph = L.ph; p.pw = L.pw; p.act = L.act; p.w_steps = L.k_pad / 16;
  p.out_lo = L.out_lo; p.R = L.out_hi - L.out_lo; p.N = L.x.n;
  const NarrowTile t = narrow_tile(L);
  p.th = t.th; p.tw = t.tw;
  p.nty = (p.R + t.th - 1) / t.th; p.ntx = (p.W_out + t.tw - 1) / t.tw;
  p.pitch = (t.tw - 1) * p.s + 3; p.ph_rows = (t.th - 1) * p.s + 3;
  p.b_first = kNoSibling;
  p.by_ntx = make_fastdiv(p.ntx); p.by_nty = make_fastdiv(p.nty); p.by_tw = small_div(t.tw);
  p.by_pitch = small_div(p.pitch); p.by_group = make_fastdiv(kGroupM * (int)gy);
  p.by_slots = make_fastdiv(p.C_in / 4 + 1);
  *gx = (unsigned)t.tiles;
  return p;
}

// Filter vectors in flight per wavefront: all of a slice of up to five or nine steps, nine of a longer one.
constexpr int kShortSteps = 5 * kWaves;
size_t patch_bytes(const NarrowParams& p) { return (size_t)p.pitch * p.ph_rows * (p.C_in * 4 + 16); }

}  // namespace

bool narrow_applies(const OpLaunch* Ls, int n) {
  if (n < 1 || n > kMaxBatch) return false;
  for (int b = 0; b < n; ++b)
    if (!narrow_shape(Ls[b])) return false;
  const long t = narrow_tiles(Ls, n);
  return t >= 1 && (t <= kTilesAlways || (t <= kTilesOverCut && !patch_applies(Ls, nullptr, n)));
}

// sibs: per band the 1 x 1 convolution that the launch computes as well, or nullptr
hipError_t launch_narrow_siblings(const OpLaunch* Ls, const OpLaunch* sibs, int n, hipStream_t s, KernelEvents* ev) {
  if (n < 1 || n > kMaxBatch) return hipErrorInvalidValue;
  const unsigned gy1 = (unsigned)((Ls[0].y.c + 15) / 16), gy2 = sibs ? (unsigned)((sibs[0].y.c + 15) / 16) : 0, gy = gy1 + gy2;
  if ((int)gy1 * 16 > conv_cout_pad(Ls[0].y.c)) return hipErrorInvalidValue;  // unguarded weight loads
  if (sibs && (!sibs[0].wd16 || (int)gy2 * 16 > conv_cout_pad(sibs[0].y.c))) return hipErrorInvalidValue;
  NarrowParams ps[kMaxBatch];
  unsigned gx[kMaxBatch];
  int m = 0;
  size_t patch = 0;
  for (int b = 0; b < n; ++b) {
    if (!narrow_shape(Ls[b])) return hipErrorInvalidValue;
    if (Ls[b].out_hi <= Ls[b].out_lo) continue;
    ps[m] = make_narrow(Ls[b], gy, &gx[m]);
    if (ps[m].th < 1 || ps[m].th * ps[m].tw > 16) return hipErrorInvalidValue;
    if (sibs) {
      const OpLaunch& q = sibs[b];
      NarrowParams& p = ps[m];
      p.b_wd16 = q.wd16; p.b_y = (float*)q.y.ptr; p.b_bias = q.bias; p.b_w_steps = q.k_pad / 16;
      p.b_y_row0 = q.y.row0; p.b_y_rows = q.y.rows; p.b_C_out = q.y.c; p.b_act = q.act;
      p.b_lo = q.out_lo; p.b_hi = q.out_hi; p.b_first = (int)gy1;
    }
    patch = std::max(patch, patch_bytes(ps[m]));
    ++m;
  }
  if (m == 0) return hipSuccess;
  const dim3 block(64 * kWaves);
  if (patch > (size_t)kMaxPatch) return hipErrorInvalidValue;
  if (patch > (size_t)kSmallPatch)
    return launch_group(conv_narrow_patch_kernel<float, 9, kMaxPatch>, conv_narrow_patch_kernel_bands<float, 9, kMaxPatch>, ps, m, gx, gy, 1, block, s, ev);
  if (9 * ps[0].C_in / 16 > kShortSteps)
    return launch_group(conv_narrow_patch_kernel<float, 9, kSmallPatch>, conv_narrow_patch_kernel_bands<float, 9, kSmallPatch>, ps, m, gx, gy, 1, block, s, ev);
  return launch_group(conv_narrow_patch_kernel<float, 5, kSmallPatch>, conv_narrow_patch_kernel_bands<float, 5, kSmallPatch>, ps, m, gx, gy, 1, block, s, ev);
}

hipError_t launch_narrow(const OpLaunch* Ls, int n, hipStream_t s, KernelEvents* ev) {
  return launch_narrow_siblings(Ls, nullptr, n, s, ev);
}
bool narrow_takes_sibling(const OpLaunch* Ls, const OpLaunch* sibs, int n) {
  return narrow_applies(Ls, n) && sibs[0].wd16 && sibs[0].y.c % 4 == 0;
}

int narrow_describe(const OpLaunch* Ls, int n, char* name, size_t size) {
  size_t patch = 0;
  int m = 0;
  for (int b = 0; b < n; ++b) {
    if (Ls[b].out_hi <= Ls[b].out_lo) continue;
    unsigned gx;
    patch = std::max(patch, patch_bytes(make_narrow(Ls[b], 1, &gx)));
    ++m;
  }
  const bool big = patch > (size_t)kSmallPatch;
  if (name && size)
    snprintf(name, size, "conv_narrow_patch_kernel%s<float, %d, %d>", m > 1 ? "_bands" : "", big || 9 * Ls[0].x.c / 16 > kShortSteps ? 9 : 5,
             big ? kMaxPatch : kSmallPatch);
  return 1;
}

}  // namespace lop
