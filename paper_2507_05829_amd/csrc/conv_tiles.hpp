// 3 x 3 convolutions by rectangles of output pixels ("tiles") and the input pixels under them ("patches"): the
// parameters of the kernels that work that way and the choice of the rectangle.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "conv_common.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

constexpr unsigned kOutside = 0x80000000u;   // a byte offset past every slab: a load from there puts zeros into LDS

// A 1 x 1 convolution of the same input with the same stride (a block's shortcut), computed by the channel tiles
// of the launch from `first` on: its weights are the centre tap of a 3 x 3 filter.
struct Sibling {
  const void* wd;
  void* y;
  const float* bias;
  int k_steps, y_row0, y_rows, C_out, act;
  int lo, hi;      // its output rows, among those of the launch
  int first;
};
constexpr int kNoSibling = 0x7fffffff;

struct PatchParams {
  const void* x;
  void* y;
  void* y2;         // second destination with y's layout, or nullptr
  const void* res;
  const void* wd;   // weights in MFMA operand order
  const void* w3;   // fp32: the same as three bf16 parts
  const float* bias;
  int x_row0, x_rows, W, C_in;
  int y_row0, y_rows, W_out, C_out;  // of the tensor that is stored (POOL: the pooled one)
  int r_row0, r_rows;
  int ph, pw, act, k_steps;          // k_steps: MFMA steps of a packed weight row
  int out_lo, R, N;                  // output rows of the convolution itself
  int Wc;                            // its columns
  int th, tw, nty, ntx;              // tile of output pixels, tiles per image in either direction
  int pitch, ph_rows;                // pixel slots per row of the patch (S == 2: even columns, then odd), its rows
  unsigned by_tw, by_pitch;          // (small_div)
  FastDiv by_ntx, by_nty, by_group;
  Sibling sib;
};
static_assert(sizeof(Batch<PatchParams>) <= 4096, "the parameters of all bands of a launch travel as kernel arguments");

// The convolution's own output rows and columns behind a launch (pooled: twice the pooled ones).
struct PatchWork { int R, Wc, N; };
inline PatchWork patch_work(const OpLaunch& c, const OpLaunch* pool) {
  if (pool) return {2 * (pool->out_hi - pool->out_lo), 2 * pool->y.w, c.x.n};
  return {c.out_hi - c.out_lo, c.y.w, c.x.n};
}

// The rectangle of at most `pixels` output pixels for R x W of them whose patch has at most `room` pixels: the
// fewest tiles, then the smallest patch, over widths that split the columns evenly.
struct PatchTile { int th = 0, tw = 0; long tiles = 0; int patch = 0; };
inline PatchTile find_tile(const PatchWork& w, int pixels, int room, int s, bool pool) {
  const int step = pool ? 2 : 1;
  PatchTile best;
  for (int target = 64; target >= 2; target /= 2) {
    const int k = (w.Wc + target - 1) / target;
    int tw = (w.Wc + k - 1) / k;
    tw = (tw + step - 1) / step * step;
    if (tw > pixels) continue;
    int th = std::min(pixels / tw, w.R) / step * step;
    const int cols = s == 1 ? tw + 2 : 2 * (tw + 1);
    while (th >= step && ((th - 1) * s + 3) * cols > room) th -= step;
    if (th < step) continue;
    const long tiles = (long)((w.R + th - 1) / th) * ((w.Wc + tw - 1) / tw) * w.N;
    const int patch = ((th - 1) * s + 3) * cols;
    if (!best.th || tiles < best.tiles || (tiles == best.tiles && patch < best.patch)) best = {th, tw, tiles, patch};
  }
  return best;
}
// (Every launch asks for the same few rectangles again and again: the last ones are remembered per thread, at places spread by
// a multiplication. A sum modulo 64 put those of one chain of twelve small bands on each other: 31 us of host time a call (2 of them the joined first layers), 26 spread.)
inline PatchTile tile_for(const PatchWork& w, int pixels, int room, int s, bool pool) {
  struct Entry { PatchWork w; int pixels, room, s; bool pool; PatchTile t; };
  thread_local Entry memo[256] = {};
  const unsigned key = ((((unsigned)w.R * 0x9e3779b1u + (unsigned)w.Wc) * 0x9e3779b1u + (unsigned)w.N) * 0x9e3779b1u + (unsigned)(pixels * 1024 + room * 4 + s * 2 + pool)) * 0x9e3779b1u;
  Entry& e = memo[key >> 24];
  if (e.w.R != w.R || e.w.Wc != w.Wc || e.w.N != w.N || e.pixels != pixels || e.room != room || e.s != s || e.pool != pool || !e.t.th)
    e = {w, pixels, room, s, pool, find_tile(w, pixels, room, s, pool)};
  return e.t;
}

inline PatchParams make_patch(const OpLaunch& c, const OpLaunch* pool, int pixels, int room, unsigned gy, unsigned* tiles) {
  PatchParams p;
  const Slab& y = pool ? pool->y : c.y;
  const PatchWork w = patch_work(c, pool);
  const int ke = c.dtype == LOP_BF16 ? 8 : 4;
  p.x = c.x.ptr; p.y = y.ptr; p.y2 = pool ? pool->y2 : c.y2; p.res = c.res.ptr; p.wd = c.wd; p.w3 = c.w3; p.bias = c.bias;
  p.x_row0 = c.x.row0; p.x_rows = c.x.rows; p.W = c.x.w; p.C_in = c.x.c;
  p.y_row0 = y.row0; p.y_rows = y.rows; p.W_out = y.w; p.C_out = c.y.c;
  p.r_row0 = c.res.row0; p.r_rows = c.res.rows;
  p.ph = c.ph; p.pw = c.pw; p.act = c.act; p.k_steps = c.k_pad / (2 * ke);
  p.out_lo = pool ? 2 * pool->out_lo : c.out_lo;
  p.R = w.R; p.N = w.N; p.Wc = w.Wc;
  const PatchTile t = tile_for(w, pixels, room, c.sh, pool != nullptr);
  p.th = t.th; p.tw = t.tw;
  p.nty = (w.R + t.th - 1) / t.th; p.ntx = (w.Wc + t.tw - 1) / t.tw;
  p.pitch = c.sh == 1 ? t.tw + 2 : 2 * (t.tw + 1);
  p.ph_rows = (t.th - 1) * c.sh + 3;
  p.by_ntx = make_fastdiv(p.ntx); p.by_nty = make_fastdiv(p.nty);
  p.by_tw = small_div(pool ? t.tw / 2 : t.tw);
  p.by_pitch = small_div(p.pitch);
  p.by_group = make_fastdiv(kGroupM * (int)gy);
  p.sib = Sibling{nullptr, nullptr, nullptr, 0, 0, 0, 0, 0, 0, 0, kNoSibling};
  *tiles = (unsigned)t.tiles;
  return p;
}

}  // namespace
}  // namespace lop
