// Two dense 3 x 3 convolutions of 16 channels, the second the only reader of the first, as one launch.
//
// Such layers are over in a few microseconds whatever the kernel: what a chain of them costs is launches (3 us of host
// time each, 4 us of a kernel that does next to nothing) and the trip of the rows between them through memory. A
// workgroup here owns 8 x 8 output pixels: the 12 x 12 input pixels under them go to LDS, the first convolution's 10 x 10
// pixels are computed from there (1.56 times the outputs: the halo of a tile is computed again by its neighbours), get bias,
// activation and the storage type's rounding, and stay in LDS for the second. Both filters are in registers before the
// first barrier (operand order of 16 x 16 tiles, a contiguous KiB per load), so there is one round of memory latency. The four
// wavefronts take the 16-pixel tiles of a layer in turn.
// It replaces two launches at every size where the pair is first or last in a chain. Between two other layers of the chain it stays
// two: the second layer's output is given the memory of the first one's input, which two launches allow and this does not.
// 16 channels only: both filters of a wavefront are 18 vectors of registers there, with 32 channels they would be 72 and
// would have to be streamed or lie in LDS. us a call (fp32, then bf16; calls in flight, and alone), two -> one: 32 x 32 pixels
// 9.1, 23 -> 4.9, 17 and 9.0, 21 -> 5.2, 16; 160 x 160 10.0, 29 -> 5.0, 19 and 9.6, 25 -> 5.0, 16; 512 x 512 84, 105 -> 30, 47 and
// 27, 49 -> 9.6, 25; 1024 x 1024 328, 357 -> 122, 145 and 107, 133 -> 40, 53. Small ones are bound by the host (a launch and
// the parameters of its bands), large fp32 ones by the fp32 matrix instructions: 1.28 times the two layers' at 128 TFLOP/s.
// The sums of a pixel are five, of 32 products at most, so that the error against 64 bits is below the two launches' (1.05e-7
// in norm against 1.20e-7).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "act.hpp"
#include "conv_common.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

constexpr int kPairC = kPairChannels, kPairTile = 8;

struct PairParams {
  const void* x;
  void* y;
  void* y2;          // second destination with y's layout, or nullptr
  const void* w1;    // weights in the operand order of 16 x 16 tiles
  const void* w2;
  const float* b1;
  const float* b2;
  int x_lo, x_hi, x_row0, x_rows;   // [x_lo, x_hi): the rows of the image that the slab holds
  int H, W;
  int y_row0, y_rows;
  int act1, act2, out_lo, R, N;
  int nty, ntx;
  FastDiv by_ntx, by_nty;
};
static_assert(sizeof(Batch<PairParams>) <= 4096, "the parameters of all bands of a launch travel as kernel arguments");

// Steps of the reduction: a filter vector of 16 bytes per lane each. fp32: a tap's 16 channels. bf16: two taps', the tenth
// tap's weights are zero in the packing.
template <typename T> constexpr int kPairSteps = sizeof(T) == 4 ? 9 : 5;

__device__ __forceinline__ f32x4 pair_mma(float, const u32x4& w, const u32x4& x, f32x4 acc) {
  const f32x4 a = __builtin_bit_cast(f32x4, w), b = __builtin_bit_cast(f32x4, x);
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
  return acc;
}
__device__ __forceinline__ f32x4 pair_mma(__bf16, const u32x4& w, const u32x4& x, f32x4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
}

// Four neighbouring channels of a pixel, activated and rounded to the storage type.
template <typename T>
struct PairOut {
  typedef unsigned raw_t __attribute__((ext_vector_type(sizeof(T))));
  static __device__ __forceinline__ raw_t make(f32x4 v, const f32x4& bias, const Clamp& cl) {
    v += bias;
    alignas(16) T o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = from_f32<T>(clamp_act(v[j], cl));
    return *(const raw_t*)o;
  }
};

template <typename T>
__device__ __forceinline__ void pair_body(const PairParams& p, const int bx) {
  constexpr int TILE = kPairTile, IN = TILE + 4, MID = TILE + 2;
  constexpr int PB = kPairC * (int)sizeof(T);          // bytes of a pixel
  constexpr int PIECES = IN * IN * PB / 16;            // 16-byte pieces of the input under a tile
  constexpr int LOADS = (PIECES + 255) / 256, STEPS = kPairSteps<T>;
  constexpr int MID_TILES = (MID * MID + 15) / 16;
  typedef PairOut<T> Out;
  // (behind the pixels of either: one of zeros, the tenth tap of bf16's last step)
  __shared__ __attribute__((aligned(16))) unsigned char in_s[(IN * IN + 1) * PB], mid_s[(MID * MID + 1) * PB];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int px = lane & 15, kq = lane >> 4;
  const int q = fastdiv(bx, p.by_ntx), tx = bx - q * p.ntx;
  const int n = fastdiv(q, p.by_nty), ty = q - n * p.nty;
  const int oh0 = p.out_lo + ty * TILE, ow0 = tx * TILE;

  // ---- everything that comes from memory
  u32x4 raw[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int piece = i * 256 + tid, pix = piece / (PB / 16), k = piece % (PB / 16);
    const int ih = oh0 - 2 + pix / IN, iw = ow0 - 2 + pix % IN;
    raw[i] = u32x4{0u, 0u, 0u, 0u};
    if (piece < PIECES && ih >= p.x_lo && ih < p.x_hi && iw >= 0 && iw < p.W)
      raw[i] = *(const u32x4*)((const char*)p.x + ((size_t)(n * p.x_rows + ih - p.x_row0) * p.W + iw) * PB + k * 16);
  }
  u32x4 w1[STEPS], w2[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) w1[s] = ((const u32x4*)p.w1)[s * 64 + lane];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) w2[s] = ((const u32x4*)p.w2)[s * 64 + lane];
  f32x4 bias1 = f32x4{0.f, 0.f, 0.f, 0.f}, bias2 = bias1;
  if (p.b1) bias1 = *(const f32x4*)(p.b1 + kq * 4);
  if (p.b2) bias2 = *(const f32x4*)(p.b2 + kq * 4);
#pragma unroll
  for (int i = 0; i < LOADS; ++i)
    if (i * 256 + tid < PIECES) *(u32x4*)(in_s + (i * 256 + tid) * 16) = raw[i];
  if (sizeof(T) == 2 && tid < PB / 16) {
    *(u32x4*)(in_s + IN * IN * PB + tid * 16) = u32x4{0u, 0u, 0u, 0u};
    *(u32x4*)(mid_s + MID * MID * PB + tid * 16) = u32x4{0u, 0u, 0u, 0u};
  }
  __syncthreads();

  // The sums of 16 pixels: this lane's operand of step s are 16 bytes of the pixel under a tap of its pixel. at: its pixel's
  // first tap; pitch: pixels per row; zeros: where the pixel of zeros lies.
  auto convolve = [&](const unsigned char* from, int at, int pitch, int zeros, const u32x4 (&w)[STEPS]) __attribute__((always_inline)) {
    f32x4 acc[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      int off;
      if constexpr (sizeof(T) == 4) {
        off = at + (s / 3 * pitch + s % 3) * PB + kq * 16;
      } else {
        const int t0 = 2 * s, t1 = 2 * s + 1;
        const int first = at + (t0 / 3 * pitch + t0 % 3) * PB, second = t1 < 9 ? at + (t1 / 3 * pitch + t1 % 3) * PB : zeros;
        off = (kq & 2 ? second : first) + (kq & 1) * 16;
      }
      acc[s % 5] = pair_mma(T{}, w[s], *(const u32x4*)(from + off), acc[s % 5]);
    }
    return ((acc[0] + acc[1]) + (acc[2] + acc[3])) + acc[4];
  };

  // ---- the first convolution, at the pixels under the tile's windows; outside the image the second one's padding
  const Clamp c1 = make_clamp(p.act1), c2 = make_clamp(p.act2);
#pragma unroll
  for (int k = 0; k < (MID_TILES + 3) / 4; ++k) {
    const int tile = wave + 4 * k;
    if (tile >= MID_TILES) continue;
    const int i = tile * 16 + px, pix = min(i, MID * MID - 1), r = pix / MID, c = pix % MID;
    const f32x4 acc = convolve(in_s, (r * IN + c) * PB, IN, IN * IN * PB, w1);
    const int mh = oh0 - 1 + r, mw = ow0 - 1 + c;
    typename Out::raw_t v = Out::make(acc, bias1, c1);
    if (mh < 0 || mh >= p.H || mw < 0 || mw >= p.W) v = typename Out::raw_t(0u);
    if (i < MID * MID) *(typename Out::raw_t*)(mid_s + pix * PB + kq * 4 * (int)sizeof(T)) = v;
  }
  __syncthreads();

  // ---- the second: one tile of 16 pixels a wavefront
  const int r = (wave * 16 + px) / TILE, c = px % TILE;
  const f32x4 acc = convolve(mid_s, (r * MID + c) * PB, MID, MID * MID * PB, w2);
  const typename Out::raw_t v = Out::make(acc, bias2, c2);
  const int oh = oh0 + r, ow = ow0 + c;
  if (oh >= p.out_lo + p.R || ow >= p.W) return;
  const size_t ya = ((size_t)(n * p.y_rows + oh - p.y_row0) * p.W + ow) * PB + kq * 4 * sizeof(T);
  *(typename Out::raw_t*)((char*)p.y + ya) = v;
  if (p.y2) *(typename Out::raw_t*)((char*)p.y2 + ya) = v;
}

template <typename T>
__global__ __launch_bounds__(256) void conv_pair_kernel(const PairParams p) {
  pair_body<T>(p, blockIdx.x);
}
// The same for several bands in one grid (band b owns blocks first[b] .. first[b + 1]).
template <typename T>
__global__ __launch_bounds__(256) void conv_pair_kernel_bands(const Batch<PairParams> t) {
  const int b = batch_find(t, blockIdx.x);
  pair_body<T>(t.p[b], blockIdx.x - t.first[b]);
}

constexpr long kPairMaxTiles = 0xffffffffL / 256;   // a launch's threads

bool pair_shape(const OpLaunch& L) {
  return L.op == LOP_CONV2D && L.wd16 && L.kh == 3 && L.kw == 3 && L.sh == 1 && L.sw == 1 && L.ph == 1 && L.pw == 1 && L.dh == 1 &&
         L.dw == 1 && L.x.c == kPairC && L.y.c == kPairC && !L.res.ptr;
}

size_t slab_bytes(const Slab& s, int dtype) { return (size_t)s.n * s.rows * s.w * s.c * (dtype == LOP_BF16 ? 2 : 4); }

// Bands whose slabs are the same tensors and whose rows follow each other are one band to this kernel, which needs
// nothing that is kept per band: fewer parameters travel (3 KB of them cost a launch 1 us on the host).
int join_bands(const OpLaunch* firsts, const OpLaunch* seconds, int n, OpLaunch* a, OpLaunch* b) {
  int m = 0;
  for (int i = 0; i < n; ++i) {
    if (seconds[i].out_hi <= seconds[i].out_lo) continue;
    if (m > 0) {
      const Slab &x = a[m - 1].x, &y = b[m - 1].y;
      if (x.ptr == firsts[i].x.ptr && x.row0 == firsts[i].x.row0 && x.rows == firsts[i].x.rows && y.ptr == seconds[i].y.ptr &&
          y.row0 == seconds[i].y.row0 && y.rows == seconds[i].y.rows && b[m - 1].out_hi == seconds[i].out_lo) {
        b[m - 1].out_hi = seconds[i].out_hi;
        continue;
      }
    }
    a[m] = firsts[i];
    b[m] = seconds[i];
    ++m;
  }
  return m;
}

long pair_tiles(const OpLaunch& L) {
  return (long)L.x.n * ((L.out_hi - L.out_lo + kPairTile - 1) / kPairTile) * ((L.y.w + kPairTile - 1) / kPairTile);
}

}  // namespace

bool pair_applies(const OpLaunch* firsts, const OpLaunch* seconds, int n) {
  if (n < 1 || n > kMaxBatch) return false;
  long tiles = 0;
  for (int b = 0; b < n; ++b) {
    if (!pair_shape(firsts[b]) || !pair_shape(seconds[b])) return false;
    if (seconds[b].out_hi > seconds[b].out_lo) tiles += pair_tiles(seconds[b]);
  }
  if (tiles > kPairMaxTiles) return false;
  // A workgroup stores its outputs while others still read their inputs: no output may lie in memory that holds an input
  // (two launches allow it, and the buffers of layers that are never needed together do share memory).
  for (int i = 0; i < n; ++i) {
    const char* const x = (const char*)firsts[i].x.ptr;
    for (int j = 0; j < n; ++j) {
      const char* const y = (const char*)seconds[j].y.ptr;
      if (x < y + slab_bytes(seconds[j].y, seconds[j].dtype) && y < x + slab_bytes(firsts[i].x, firsts[i].dtype)) return false;
    }
  }
  return true;
}

hipError_t launch_pair(const OpLaunch* firsts, const OpLaunch* seconds, int n, hipStream_t stream, KernelEvents* ev) {
  if (!pair_applies(firsts, seconds, n)) return hipErrorInvalidValue;
  OpLaunch as[kMaxBatch], bs[kMaxBatch];
  const int m = join_bands(firsts, seconds, n, as, bs);
  PairParams ps[kMaxBatch];
  unsigned gx[kMaxBatch];
  for (int i = 0; i < m; ++i) {
    const OpLaunch &a = as[i], &b = bs[i];
    PairParams& p = ps[i];
    p.x = a.x.ptr; p.y = b.y.ptr; p.y2 = b.y2;
    p.w1 = a.wd16; p.w2 = b.wd16; p.b1 = a.bias; p.b2 = b.bias;
    p.x_lo = std::max(0, a.x.row0); p.x_hi = std::min(a.x.h, a.x.row0 + a.x.rows); p.x_row0 = a.x.row0; p.x_rows = a.x.rows;
    p.H = a.x.h; p.W = a.x.w;
    p.y_row0 = b.y.row0; p.y_rows = b.y.rows;
    p.act1 = a.act; p.act2 = b.act; p.out_lo = b.out_lo; p.R = b.out_hi - b.out_lo; p.N = a.x.n;
    p.nty = (p.R + kPairTile - 1) / kPairTile; p.ntx = (p.W + kPairTile - 1) / kPairTile;
    p.by_ntx = make_fastdiv(p.ntx); p.by_nty = make_fastdiv(p.nty);
    gx[i] = (unsigned)pair_tiles(b);
  }
  if (m == 0) return hipSuccess;
  const dim3 block(256);
  return as[0].dtype == LOP_BF16 ? launch_group(conv_pair_kernel<__bf16>, conv_pair_kernel_bands<__bf16>, ps, m, gx, 1, 1, block, stream, ev)
                                 : launch_group(conv_pair_kernel<float>, conv_pair_kernel_bands<float>, ps, m, gx, 1, 1, block, stream, ev);
}

}  // namespace lop
