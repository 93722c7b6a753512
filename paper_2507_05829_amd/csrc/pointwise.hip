// 1x1 stride-1 convolution = the row-wise local operator (Intra-DP Sec. IV-A, Eq. 1): every
// output pixel is its own input row times the whole weight matrix, so a row band needs no
// halo at all. With few channels this is a bandwidth-bound stream, not a GEMM to tile: a
// wavefront takes 32 pixels, loads their channels straight from global memory in the operand
// layout (no LDS staging) and the entire weight matrix as MFMA operand fragments (which the 16 wavefronts
// of a compute unit find in the vector cache), multiplies, and turns the accumulators, two tiles of 32
// channels at a time, through a small wave-private LDS region so that every store and residual load is a
// contiguous 16-byte piece per lane. All loads of a wavefront are issued before its first store: on this
// architecture loads and stores share one in-order counter, so a load waited for after a
// store would also wait for the store to be acknowledged.
// What bounds it is memory, and that a launch of some ten microseconds starts and ends with the chip idle: hence the
// accumulators of two tiles at a time only, the bias in LDS and one group of pixels a wavefront, which makes four
// wavefronts per SIMD where accumulators of all tiles and two groups made two (32 -> 192 channels on 130 000 pixels,
// 61 MB, 19.9 -> 15.8 us; on 30 000 9.7 -> 7.9). A large launch takes four groups a wavefront, whose weights are then
// loaded once: on 550 000 pixels, 245 MB, 52.5 us against 59 with one.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>

#include "act.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct PwParams {
  const __bf16* x;
  __bf16* y;
  const __bf16* res;
  const __bf16* w;  // [c_out_pad][k_pad]
  const float* bias;
  int x_row0, x_rows, W, C_in;
  int y_row0, y_rows, C_out;
  int r_row0, r_rows;
  int act, out_lo, R, N;
  int M;  // N * R * W
  int k_pad;
  int groups;  // ceil(M / 32)
};
static_assert(sizeof(Batch<PwParams>) <= 4096, "the parameters of all bands of a launch travel as kernel arguments");

// The staging rows are private to a wavefront and the LDS executes one wavefront's
// instructions in issue order, so a write followed by a read of another lane's data needs
// no barrier: only the compiler has to be kept from reordering the two.
__device__ __forceinline__ void lds_wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// NT: 32-channel tiles of the output (C_out = 32 * NT); KS: 16-element steps of the
// reduction (C_in = 16 * KS); RES: a residual is added (its loads are the only loads
// issued after the first store; without it the store stream is never waited for).
template <int NT, int KS, bool RES, int GPW>
__device__ __forceinline__ void pointwise_body(const PwParams& p, const int bx) {
  constexpr int CH = NT >= 2 ? 2 : 1;   // tiles turned through LDS at a time
  constexpr int CP = CH * 32 + 4;       // fp32 pitch of the staged rows
  __shared__ __attribute__((aligned(16))) float stage[4][32 * CP + NT * 32];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int px = lane & 31, kg = lane >> 5;
  float* const st = stage[wave];
  float* const bias = st + 32 * CP;
  const Clamp clamp = make_clamp(p.act);
  const int first = (bx * 4 + wave) * GPW;
  if (first >= p.groups) return;

  // A band of a 1x1 stride-1 layer is one contiguous run of pixels per image in the input,
  // output and residual slabs alike, so a pixel's address is linear in its index m once
  // the image n = m / (R*W) is known: off(m) = (n*img + first + (m - n*R*W)) * channels.
  const int RW = p.R * p.W;
  const long x_img = (long)p.x_rows * p.W, x_first = (long)(p.out_lo - p.x_row0) * p.W;
  const long y_img = (long)p.y_rows * p.W, y_first = (long)(p.out_lo - p.y_row0) * p.W;
  const long r_img = (long)p.r_rows * p.W, r_first = (long)(p.out_lo - p.r_row0) * p.W;

  // a group's first pixel and its image: one division (wave-uniform); pixel m0 + q lies wraps(q) images further (at most
  // one when an image's band holds at least 32 pixels)
  int m0, n0, rem0;
  auto place = [&](int g) __attribute__((always_inline)) { m0 = g * 32; n0 = m0 / RW; rem0 = m0 - n0 * RW; };
  auto wraps = [&](int q) { return RW >= 32 ? (rem0 + q >= RW ? 1 : 0) : (rem0 + q) / RW; };

  uint4 x[GPW][KS];
#pragma unroll
  for (int i = 0; i < GPW; ++i) {
    place(first + i);
    if (m0 + px < p.M) {
      const __bf16* src = p.x + (size_t)(n0 * x_img + x_first + rem0 + px + wraps(px) * (x_img - RW)) * p.C_in + kg * 8;
#pragma unroll
      for (int s = 0; s < KS; ++s) x[i][s] = *(const uint4*)(src + s * 16);
    } else {
#pragma unroll
      for (int s = 0; s < KS; ++s) x[i][s] = make_uint4(0, 0, 0, 0);
    }
  }
  // the whole weight matrix as A-operand fragments: tile t, step s -> channels t*32+px,
  // reduction elements s*16 + kg*8 .. +8
  uint4 wf[NT][KS];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int s = 0; s < KS; ++s)
      wf[t][s] = *(const uint4*)(p.w + (size_t)(t * 32 + px) * p.k_pad + s * 16 + kg * 8);
  float bv[(NT + 1) / 2];
#pragma unroll
  for (int i = 0; i < (NT + 1) / 2; ++i) bv[i] = p.bias && i * 64 + lane < NT * 32 ? p.bias[i * 64 + lane] : 0.f;
#pragma unroll
  for (int i = 0; i < (NT + 1) / 2; ++i)
    if (i * 64 + lane < NT * 32) bias[i * 64 + lane] = bv[i];
  // Every load above is waited for here, before the first store is issued.
#pragma unroll
  for (int i = 0; i < GPW; ++i)
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" ::"v"(x[i][s].x), "v"(x[i][s].y), "v"(x[i][s].z), "v"(x[i][s].w));
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" ::"v"(wf[t][s].x), "v"(wf[t][s].y), "v"(wf[t][s].z), "v"(wf[t][s].w));

  constexpr int TURNS = (NT + CH - 1) / CH;
#pragma unroll
  for (int i = 0; i < GPW; ++i) {
  place(first + i);
#pragma unroll
  for (int tu = 0; tu < TURNS; ++tu) {
    const int c0 = tu * CH;
    const int tiles = (NT - c0) < CH ? (NT - c0) : CH;
    f32x16 acc[CH];
#pragma unroll
    for (int t = 0; t < CH; ++t)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[t][k] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int t = 0; t < CH; ++t)
        if (c0 + t < NT)
          acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[c0 + t][s]),
                                                           __builtin_bit_cast(bf16x8, x[i][s]), acc[t], 0, 0, 0);

    // ---- epilogue of the turn's 32*CH channels through this wave's LDS rows.
    // Accumulator layout: pixel px, channels g8*8 + kg*4 + {0..3} of the tile, g8 = 0..3.
    // In a turn of `tiles` tiles a pixel has VPP = 4*tiles 16-byte pieces; lane owns piece v = lane % VPP of
    // pixels q = lane / VPP + j * (64 / VPP).
    const int VPP = tiles * 4, QSTEP = 64 / VPP;
    lds_wave_order();  // the previous turn's reads are issued before these writes
#pragma unroll
    for (int t = 0; t < CH; ++t) {
      if (c0 + t < NT) {
#pragma unroll
        for (int g8 = 0; g8 < 4; ++g8)
          *(float4*)(st + px * CP + t * 32 + g8 * 8 + kg * 4) =
              make_float4(acc[t][g8 * 4], acc[t][g8 * 4 + 1], acc[t][g8 * 4 + 2], acc[t][g8 * 4 + 3]);
      }
    }
    lds_wave_order();
    const int v = lane % VPP, q0 = lane / VPP;
    float bb[8];
    *(float4*)bb = *(const float4*)(bias + c0 * 32 + v * 8);
    *(float4*)(bb + 4) = *(const float4*)(bias + c0 * 32 + v * 8 + 4);
    // Addresses: one wave-uniform base plus a 32-bit per-lane offset; each image a pixel lies further adds
    // (img - R*W) pixels of rows outside the band.
    __bf16* const ybase = p.y + ((size_t)n0 * y_img + y_first + rem0) * p.C_out + c0 * 32 + v * 8;
    const __bf16* const rbase =
        RES ? p.res + ((size_t)n0 * r_img + r_first + rem0) * p.C_out + c0 * 32 + v * 8 : nullptr;
    constexpr int JN = 32 / (64 / ((CH < 2 ? 1 : 2) * 4));  // upper bound of slots per lane
    uint4 rres[JN];
    if constexpr (RES) {
#pragma unroll
      for (int j = 0; j < 32 / QSTEP; ++j) {
        const int q = q0 + j * QSTEP;
        rres[j] = make_uint4(0, 0, 0, 0);
        if (m0 + q < p.M) rres[j] = *(const uint4*)(rbase + (q + wraps(q) * (int)(r_img - RW)) * p.C_out);
      }
      // one wait for the turn's residual vectors
#pragma unroll
      for (int j = 0; j < 32 / QSTEP; ++j) asm volatile("" ::"v"(rres[j].x), "v"(rres[j].y), "v"(rres[j].z), "v"(rres[j].w));
    }
#pragma unroll
    for (int j = 0; j < 32 / QSTEP; ++j) {
      const int q = q0 + j * QSTEP;
      if (m0 + q >= p.M) continue;
      const float4 lo = *(const float4*)(st + q * CP + v * 8);
      const float4 hi = *(const float4*)(st + q * CP + v * 8 + 4);
      float o[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] += bb[i];
      if constexpr (RES) {
        const unsigned u[4] = {rres[j].x, rres[j].y, rres[j].z, rres[j].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          o[2 * i] += __uint_as_float(u[i] << 16);
          o[2 * i + 1] += __uint_as_float(u[i] & 0xffff0000u);
        }
      }
      alignas(16) __bf16 ob[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) ob[i] = (__bf16)clamp_act(o[i], clamp);
      *(uint4*)(ybase + (q + wraps(q) * (int)(y_img - RW)) * p.C_out) = *(const uint4*)ob;
    }
  }
  }
}

template <int NT, int KS, bool RES, int GPW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void pointwise_kernel(const PwParams p) {
  pointwise_body<NT, KS, RES, GPW>(p, blockIdx.x);
}
// The same for several bands of one layer in one grid (band b owns blocks first[b] .. first[b + 1]).
template <int NT, int KS, bool RES, int GPW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void pointwise_kernel_bands(const Batch<PwParams> t) {
  const int b = batch_find(t, blockIdx.x);
  pointwise_body<NT, KS, RES, GPW>(t.p[b], blockIdx.x - t.first[b]);
}

template <int NT, int KS, int GPW>
hipError_t launch_pw(const PwParams* ps, int n, hipStream_t s, KernelEvents* ev) {
  unsigned gx[kMaxBatch];
  for (int b = 0; b < n; ++b) gx[b] = (unsigned)((ps[b].groups + 4 * GPW - 1) / (4 * GPW));
  if constexpr (GPW == 1) {
    if (ps[0].res) return launch_group(pointwise_kernel<NT, KS, true, 1>, pointwise_kernel_bands<NT, KS, true, 1>, ps, n, gx, 1, 1, dim3(256), s, ev);
  }
  return launch_group(pointwise_kernel<NT, KS, false, GPW>, pointwise_kernel_bands<NT, KS, false, GPW>, ps, n, gx, 1, 1, dim3(256), s, ev);
}

// Groups of pixels a wavefront takes: four in launches of many (short reductions: their inputs are all in registers at
// once). Four a wavefront below, us a launch of 32 -> 192 channels: 4 100 groups 18.7 against 15.8, 3 700 15.2 against 14.1.
// One with a residual, whose loads the four would wait for one group after the other (32 -> 192 with four also
// spills): 25 600 groups 32 -> 192 136 us with one, 145 with four, 32 -> 64 41 and 45, 32 -> 32 24.3 and 24.4; 9 100 42 and 49, 17.0 and 17.6, 10.3 and 12.0.
constexpr long kManyGroups = 8192;
long pw_groups(const OpLaunch& L) { return ((long)L.x.n * std::max(0, L.out_hi - L.out_lo) * L.x.w + 31) / 32; }
int pw_groups_per_wavefront(const OpLaunch* Ls, int n, int ks) {
  long groups = 0;
  for (int b = 0; b < n; ++b) groups += pw_groups(Ls[b]);
  return ks <= 2 && !Ls[0].res.ptr && groups >= kManyGroups ? 4 : 1;
}

struct PwShape { int nt, ks; };
constexpr PwShape kPwShapes[] = {{6, 2}, {1, 12}, {1, 2}, {2, 2}, {4, 2}, {1, 4}, {2, 4}, {4, 4}, {1, 8}, {2, 8}};

bool pw_find(const OpLaunch& L, int* nt, int* ks) {
  if (L.op != LOP_CONV2D || L.dtype != LOP_BF16) return false;
  if (L.kh != 1 || L.kw != 1 || L.sh != 1 || L.sw != 1 || L.ph != 0 || L.pw != 0) return false;
  if (L.x.c % 16 != 0 || L.y.c % 32 != 0) return false;
  *nt = L.y.c / 32;
  *ks = L.x.c / 16;
  for (const PwShape& sh : kPwShapes)
    if (sh.nt == *nt && sh.ks == *ks) return true;
  return false;
}

}  // namespace

// True when the bandwidth-bound 1x1 kernel takes this launch instead of the implicit GEMM.
bool pointwise_applies(const OpLaunch& L) {
  int nt, ks;
  return pw_find(L, &nt, &ks);
}

int pointwise_describe(const OpLaunch* Ls, int n, char* name, size_t size) {
  int nt = 0, ks = 0, m = 0;
  pw_find(Ls[0], &nt, &ks);
  for (int b = 0; b < n; ++b) m += Ls[b].out_hi > Ls[b].out_lo;
  if (name && size)
    snprintf(name, size, "pointwise_kernel%s<%d, %d, %s, %d>", m > 1 ? "_bands" : "", nt, ks, Ls[0].res.ptr ? "true" : "false",
             pw_groups_per_wavefront(Ls, n, ks));
  return 1;
}

hipError_t launch_pointwise(const OpLaunch* Ls, int n, hipStream_t stream, KernelEvents* ev) {
  int nt = 0, ks = 0, m = 0;
  if (n < 1 || n > kMaxBatch || !pw_find(Ls[0], &nt, &ks)) return hipErrorInvalidValue;
  const int per = pw_groups_per_wavefront(Ls, n, ks);
  PwParams ps[kMaxBatch];
  for (int b = 0; b < n; ++b) {
    const OpLaunch& L = Ls[b];
    PwParams& p = ps[m];
    p.x = (const __bf16*)L.x.ptr; p.y = (__bf16*)L.y.ptr; p.res = (const __bf16*)L.res.ptr;
    p.w = (const __bf16*)L.w; p.bias = L.bias;
    p.x_row0 = L.x.row0; p.x_rows = L.x.rows; p.W = L.x.w; p.C_in = L.x.c;
    p.y_row0 = L.y.row0; p.y_rows = L.y.rows; p.C_out = L.y.c;
    p.r_row0 = L.res.row0; p.r_rows = L.res.rows;
    p.act = L.act; p.out_lo = L.out_lo; p.R = L.out_hi - L.out_lo; p.N = L.x.n;
    p.M = p.N * p.R * p.W;
    p.k_pad = L.k_pad;
    p.groups = (int)pw_groups(L);
    if (p.M > 0) ++m;
  }
  if (m == 0) return hipSuccess;
#define LOP_PW_CASE(NT, KS) if (nt == NT && ks == KS) return per == 4 ? launch_pw<NT, KS, KS <= 2 ? 4 : 1>(ps, m, stream, ev) : launch_pw<NT, KS, 1>(ps, m, stream, ev)
  LOP_PW_CASE(6, 2); LOP_PW_CASE(1, 12); LOP_PW_CASE(1, 2); LOP_PW_CASE(2, 2); LOP_PW_CASE(4, 2);
  LOP_PW_CASE(1, 4); LOP_PW_CASE(2, 4); LOP_PW_CASE(4, 4); LOP_PW_CASE(1, 8); LOP_PW_CASE(2, 8);
#undef LOP_PW_CASE
  return hipErrorInvalidValue;
}

}  // namespace lop
