// Inverted-residual block in one launch: 1x1 expand + activation, depthwise 3x3 (stride 1 or 2)
// + activation, 1x1 project (+ residual), on a row interval of the block's output.
//
// The three operators are local (Intra-DP Sec. IV-A: a block-wise operator between two
// row-wise ones, Eq. 1), so a tile of the block's output depends on a slightly larger tile of
// its input only. Run layer by layer the expanded tensor (6x the channels) is written to HBM
// and read back twice; here it never leaves the compute unit. A workgroup owns 8 x 16
// output pixels (16 x 16 in large launches of stride 1: see mb_rows) and walks over the expanded channels in chunks of 32, all three operators on the
// matrix cores:
//   expand   16 x 16 x 32 products (the whole reduction in one), pixels as rows, so that a lane ends with four neighbouring
//            pixels of one channel; 16 pixels' instructions run under the vector instructions of the 16 before them
//            (32 x 32 x 16 products tile by tile -> these: eight images of 640 x 640 through six blocks, eight bands with
//            shared rows, 505 -> 494 us alone, 393 -> 379 in flight) -> bias, activation, one rounding to bf16 -> LDS, channel by channel. Pixels
//            outside the image are zero there (the depthwise operator pads its input, i.e. the
//            expanded tensor, not the block's input);
//   depthwise  4 x 4 x 4 products, 16 channels at once, one per block of the instruction: four
//            output columns x four output rows, the reduction running over four neighbouring input
//            columns, whose weights form a band of a small matrix (one per filter row and group of
//            columns; packed behind the operator's weights). Six of them make 16 outputs of 16
//            channels (stride 2: nine) -> bias, activation, one rounding -> LDS, channel by channel,
//            from where the projection reads it transposed;
//   project  32 x 32 x 16 products: adds the chunk's contribution to the 32 output channels
//            (accumulators stay in registers over the chunks).
// What bounds it: a wavefront's instructions one after another, with three wavefronts on a SIMD (LDS holds no more): the vector
// ALUs are busy half of the time, LDS a little more, the vector cache half, the matrix cores a quarter. Leaving out one
// kind saves its share: the weights' loads 13 %, the projection 9, the depthwise products 6, the activations of the
// expanded values 5, the barriers 2. Weights are read in the
// order of the lanes, straight from the cache; barriers wait for LDS only, so that the next chunk's weights
// stay in flight; rows and channels lie in LDS in an order that has no bank conflicts; the projection's operands come out of LDS
// while the next chunk is expanded (with this and no bounds to check away from the borders the same chain takes
// 480 us alone instead of 494, 375 in flight instead of 379). What came
// before: diagonal 32 x 32 x 16 products for the depthwise part (three times the matrix cycles, diagonals
// built on the vector ALUs); weights read row by row, four cache lines per four lanes, cost a quarter more.
// The roundings are the ones the layer-by-layer path makes, so results agree with it to fp32
// summation order. Shapes: 32 input and 32 output channels, up to 192 expanded channels, bf16.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <type_traits>

#include "act.hpp"
#include "conv_common.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "lop.h"

namespace lop {
namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kMbC = 32;          // input and output channels
constexpr int kMbMaxMid = 192;    // expanded channels held by the staged biases

struct MbParams {
  const __bf16* x;
  __bf16* y;
  const __bf16* res;
  const void* we;     // expand weights in the operand order of 16 x 16 tiles, a tile of 16 channels every ke_pad / 32 steps
  const float* be;
  const void* bands;  // depthwise weights as bands (mbconv_pack_bands)
  const float* bd;
  const void* wp;     // project weights in operand order
  const float* bp;
  int e_steps;
  int x_row0, x_rows, H, W;
  int y_row0, y_rows, W_out;
  int r_row0, r_rows;
  int C_mid, nch;
  Clamp ce, cd, cp;
  int out_lo, R, N;
  int tiles_x, tiles_y;
  FastDiv by_tx, by_ty;
};

__device__ __forceinline__ f32x16 mma_bf16(const u32x4& a, const u32x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mma16_bf16(const u32x4& a, const u32x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// four bf16 (8 bytes) <-> four floats
__device__ __forceinline__ void unpack4(const u32x2& v, float* f) {
  f[0] = __builtin_bit_cast(float, v.x << 16);
  f[1] = __builtin_bit_cast(float, v.x & 0xffff0000u);
  f[2] = __builtin_bit_cast(float, v.y << 16);
  f[3] = __builtin_bit_cast(float, v.y & 0xffff0000u);
}
__device__ __forceinline__ u32x2 pack4(const float* f) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 b;
  b[0] = (__bf16)f[0]; b[1] = (__bf16)f[1]; b[2] = (__bf16)f[2]; b[3] = (__bf16)f[3];
  return __builtin_bit_cast(u32x2, b);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));

// Of 16 lanes, lane i gets value i % 4 of the four that lanes i / 4, i / 4 + 4, + 8 and + 12 point at.
__device__ __forceinline__ u32x2 transposed_read(const unsigned char* at) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)at));
}

template <int S, int ROWS>
struct MbTile {
  static constexpr int TH = ROWS, TW = 16;               // output pixels of a workgroup
  static constexpr int EH = (TH - 1) * S + 3;            // rows of expanded pixels it needs
  static constexpr int XQ = S == 1 ? 5 : 9;              // columns, in groups ("quads") of four
  static constexpr int NQ = EH * XQ;                     // quads, column of quads by column
  static constexpr int MT_E = (NQ + 7) / 8;              // expand MFMA tiles
  static constexpr int MPW = (MT_E + 3) / 4;             // ... per wavefront
  static constexpr int OP = TH * TW;
  static constexpr int RG = TH / 8;                      // groups of 8 rows: MFMA tiles of the output per wavefront
  static constexpr int KS = S == 1 ? 2 : 3;              // quads of input columns under four outputs
  // Bytes of a channel in LDS: an odd multiple of 8, which with the order of rows and channels below
  // lets every half wavefront's access touch each bank once.
  static constexpr int EPITCH = MT_E * 64 + 8;
  static constexpr int DPITCH = OP * 2 + 8;
  // The quads of an expand tile's eight that 16 pixels of it (half h) are, in the order of the operand's rows: two that half a
  // wavefront stores at once lie four apart, which with 16 channels each touches every bank of LDS once.
  __host__ __device__ static constexpr int quad(int h, int j) { return 2 * h + (j >> 1) + 4 * (j & 1); }
  // Row of the idx-th quad of a column: with stride 2 the even rows first, so that the rows under
  // neighbouring output rows are neighbours.
  __host__ __device__ static constexpr int row(int idx) { return S == 1 ? idx : idx <= TH ? 2 * idx : 2 * (idx - TH) - 1; }
  __host__ __device__ static constexpr int tap_row(int a) { return S == 1 ? a : a == 1 ? TH + 1 : a / 2; }
};

// Channel (of a chunk's 32) kept in slot s of LDS. The order is the one in which a lane's eight
// reduction values of the projection, which it reads from slots 8 j + 4 h + 2 u + kg, are
// consecutive channels.
__host__ __device__ constexpr int slot_channel(int s) {
  return ((s >> 2) & 1) * 16 + (s & 1) * 8 + ((s >> 1) & 1) * 4 + (s >> 3);
}
__host__ __device__ constexpr int channel_slot(int c) { return (c & 3) * 8 + (c >> 4) * 4 + ((c >> 2) & 1) * 2 + ((c >> 3) & 1); }
// Slot of the depthwise operator's block of lanes (lane / 4) and half of the channels.
__host__ __device__ constexpr int dw_slot(int block, int half) { return 4 * (block & 7) + 2 * half + (block >> 3); }

template <int S, bool RES, int ROWS>
__device__ __forceinline__ void mbconv_body(const MbParams& p, int bid) {
  typedef MbTile<S, ROWS> G;
  constexpr int TH = G::TH, TW = G::TW, EH = G::EH, XQ = G::XQ, NQ = G::NQ, MT_E = G::MT_E, MPW = G::MPW, KS = G::KS, RG = G::RG;
  constexpr int EPITCH = G::EPITCH, DPITCH = G::DPITCH;
  static_assert(TH == 8 || TH == 16, "groups of 8 rows");
  static_assert(NQ <= 256 && kMbMaxMid <= 256, "a thread per quad and per bias");
  __shared__ __attribute__((aligned(16))) unsigned char E_s[32 * EPITCH];   // [slot][quad]
  __shared__ __attribute__((aligned(16))) unsigned char D_s[32 * DPITCH];   // [slot][column of quads][row]
  __shared__ __attribute__((aligned(16))) float bias_s[2][kMbMaxMid];       // expand, depthwise
  __shared__ u32x2 mask_s[MT_E * 8];                                        // bits of a quad inside the image

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int px = lane & 31, kg = lane >> 5;
  const int row = fastdiv(bid, p.by_tx), tx = bid - row * p.tiles_x;
  const int n = fastdiv(row, p.by_ty), ty = row - n * p.tiles_y;
  const int oh0 = p.out_lo + ty * TH, ow0 = tx * TW;
  const int ih_base = oh0 * S - 1, iw_base = ow0 * S - 1;
  // rows of the image that the slab holds
  const int ih_lo = max(0, p.x_row0), ih_hi = min(p.H, p.x_row0 + p.x_rows);

  // A tile away from the image's borders needs no masks.
  const bool inside = ih_base >= ih_lo && iw_base >= 0 && ih_base + EH <= ih_hi && iw_base + XQ * 4 <= p.W;

  // ---- the block's input at the expanded pixels of this wavefront's MFMA tiles, in operand
  // layout (lane = pixel, eight of its channels), kept for all chunks. (Quads past the last are that one again: their memory
  // in LDS is nobody's.)
  u32x4 xa[MPW][2];
  {
    const char* const origin = (const char*)(p.x + ((long)(n * p.x_rows + ih_base - p.x_row0) * p.W + iw_base) * kMbC);
    const unsigned pitch = (unsigned)p.W * (kMbC * 2), lane_at = (lane & 3) * (kMbC * 2) + (lane >> 4) * 16;
    const int q0 = wave * 8 + G::quad(0, (lane & 15) >> 2);
    auto load = [&](auto all) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < MPW; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int q = min(q0 + 32 * i + 2 * h, NQ - 1), qx = q / EH, r = G::row(q - qx * EH);
          const u32x4* const at = (const u32x4*)(origin + ((unsigned long)(unsigned)r * pitch + qx * (kMbC * 8) + lane_at));
          if constexpr (all) {
            xa[i][h] = *at;
          } else {
            const int ih = ih_base + r, iw = iw_base + qx * 4 + (lane & 3);
            xa[i][h] = u32x4{0u, 0u, 0u, 0u};
            if (ih >= ih_lo && ih < ih_hi && iw >= 0 && iw < p.W) xa[i][h] = *at;
          }
        }
    };
    if (inside) load(std::true_type{});
    else load(std::false_type{});
  }

  // weights of a chunk: expand, the depthwise bands of this wavefront's 16 channels, project, all in the order of the
  // lanes (an access of four lanes to one 64-byte line each costs the vector cache four times as much); each part is fetched for the next chunk when this one is done with it
  const int chalf = wave & 1, rgroup = wave >> 1;          // depthwise: 16 channels x 4 rows of every 8 x 16 columns each
  u32x4 we[2], wp[2];
  s16x4 wd[3 * KS];
  const u32x4* const we_at = (const u32x4*)p.we + lane;
  const u32x4* const wp_at = (const u32x4*)p.wp + lane;
  const s16x4* const wd_at = (const s16x4*)p.bands + chalf * (3 * KS * 64) + lane;
  auto fetch_expand = [&](int c) __attribute__((always_inline)) {
    we[0] = we_at[(size_t)(2 * c) * p.e_steps * 64];
    we[1] = we_at[(size_t)(2 * c + 1) * p.e_steps * 64];
  };
  auto fetch_depthwise = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 3 * KS; ++t) wd[t] = wd_at[c * (2 * 3 * KS * 64) + t * 64];
  };
  auto fetch_project = [&](int c) __attribute__((always_inline)) {
    wp[0] = wp_at[c * 128];
    wp[1] = wp_at[c * 128 + 64];
  };
  fetch_expand(0);
  fetch_depthwise(0);
  fetch_project(0);

  if (tid < kMbMaxMid) {
    const bool in = tid < p.C_mid;
    bias_s[0][tid] = in && p.be ? p.be[tid] : 0.f;
    bias_s[1][tid] = in && p.bd ? p.bd[tid] : 0.f;
  }
  if (!inside && tid < MT_E * 8) {
    const int qx = tid / EH, ih = ih_base + G::row(tid - qx * EH), iw = iw_base + qx * 4;
    const bool rows = ih >= ih_lo && ih < ih_hi;
    auto in = [&](int k) { return rows && iw + k >= 0 && iw + k < p.W; };
    mask_s[tid] = u32x2{(in(0) ? 0xffffu : 0u) | (in(1) ? 0xffff0000u : 0u), (in(2) ? 0xffffu : 0u) | (in(3) ? 0xffff0000u : 0u)};
  }
  // LDS barrier that leaves the weights in flight alone
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  barrier();

  f32x16 acc[RG];
#pragma unroll
  for (int g = 0; g < RG; ++g)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[g][i] = 0.f;

  // expand: stores to the slot of channel px; depthwise: row lane % 4 of this wavefront's four, channel slot of its block of
  // lanes; project: a transposing read gives the lane four slots of its pixel (16 lanes read 4 slots x 4 quads)
  unsigned char* const eout = E_s + channel_slot(lane & 15) * EPITCH + (wave * 8 + G::quad(0, lane >> 4)) * 8;
  static_assert(channel_slot(16) == 4 && channel_slot(31) == channel_slot(15) + 4, "the second 16 channels lie 4 slots further");
  const int dslot = dw_slot(lane >> 2, chalf), drow = rgroup * 4 + (lane & 3);
  const unsigned char* const ewin = E_s + dslot * EPITCH + drow * 8;
  unsigned char* const dout = D_s + dslot * DPITCH + drow * 8;
  unsigned char* const dtr = D_s + (((lane & 15) >> 2) * 8 + kg) * DPITCH + (wave * RG * 8 + ((lane >> 4) & 1) * 4 + (lane & 3)) * 8;

  // ---- expand: chunk c, whose weights are in `we`
  auto expand_chunk = [&](int c, auto&& meanwhile) __attribute__((always_inline)) {
    f32x4 ebias[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float eb = bias_s[0][c * 32 + t * 16 + (lane & 15)];
      ebias[t] = f32x4{eb, eb, eb, eb};
    }
    // units of 16 pixels x 32 channels
    auto multiply = [&](int u, f32x4 (&a)[2]) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < 2; ++t) a[t] = mma16_bf16(xa[u / 2][u % 2], we[t], ebias[t]);
    };
    auto finish = [&](int u, const f32x4 (&a)[2], auto masked) __attribute__((always_inline)) {
      if (MT_E % 4 != 0 && u / 2 == MPW - 1 && wave + 4 * (u / 2) >= MT_E) return;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = clamp_act(a[t][k], p.ce);
        u32x2 pk = pack4(v);
        if constexpr (masked) pk &= mask_s[(wave + 4 * (u / 2)) * 8 + G::quad(u % 2, lane >> 4)];   // padding of the depthwise operator
        *(u32x2*)(eout + t * 4 * EPITCH + (u / 2 * 32 + u % 2 * 2) * 8) = pk;
      }
    };
    // (a tile's matrix instructions run under the vector instructions of the one before it; the branch on `inside` around all
    // of them, not in each: blocks of code are scheduled one by one)
    auto expand = [&](auto masked) __attribute__((always_inline)) {
      f32x4 a[2][2];
      multiply(0, a[0]);
#pragma unroll
      for (int u = 0; u < 2 * MPW; ++u) {
        if (u + 1 < 2 * MPW) multiply(u + 1, a[(u + 1) & 1]);
        finish(u, a[u & 1], masked);
        if (u == 1) meanwhile();
        __builtin_amdgcn_sched_barrier(0);   // (all tiles' sums at once do not fit the registers)
      }
    };
    if (inside) expand(std::false_type{});
    else expand(std::true_type{});
  };
  expand_chunk(0, [] {});
  for (int c = 0; c < p.nch; ++c) {
    const int cn = min(c + 1, p.nch - 1);
    fetch_expand(cn);
    barrier();

    // ---- depthwise 3x3 on the chunk
    {
      const float db = bias_s[1][c * 32 + slot_channel(dslot)];
      const f32x4 dbias = f32x4{db, db, db, db};
#pragma unroll
      for (int r = 0; r < RG; ++r) {
        f32x4 d[4];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          s16x4 col[XQ];
#pragma unroll
          for (int x = 0; x < XQ; ++x) col[x] = *(const s16x4*)(ewin + (x * EH + G::tap_row(a) + r * 8) * 8);
#pragma unroll
          for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int b = 0; b < 4; ++b)
              d[b] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(wd[a * KS + s], col[b * S + s], a + s ? d[b] : dbias, 0, 0, 0);
        }
        if (r == RG - 1) fetch_depthwise(cn);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          float v[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = clamp_act(d[b][k], p.cd);
          *(u32x2*)(dout + (b * TH + r * 8) * 8) = pack4(v);
        }
        if (RG > 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
    barrier();

    // ---- project: this chunk's 32 channels are the reduction axis. Its operands come out of LDS while the next chunk is
    // expanded.
    u32x2 d[RG][2][2];
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 2; ++k) d[g][h][k] = transposed_read(dtr + (4 * h + 2 * k) * DPITCH + g * 64);
    __builtin_amdgcn_sched_barrier(0);
    auto project = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[g] = mma_bf16(wp[h], u32x4{d[g][h][0].x, d[g][h][0].y, d[g][h][1].x, d[g][h][1].y}, acc[g]);
    };
    if constexpr (S == 2) {   // (with stride 2 the operands have to make room for the rest of the expand part)
      if (c + 1 < p.nch) expand_chunk(c + 1, project);
      else project();
    } else {
      if (c + 1 < p.nch) expand_chunk(c + 1, [] {});
      project();
    }
    fetch_project(cn);
  }

  // ---- bias, residual, activation, the one rounding. A lane has channels 8 g + 4 kg + {0..3} of its
  // pixel; two groups are exchanged between the lane halves so that each has 8 consecutive ones.
#pragma unroll
  for (int t = 0; t < RG; ++t) {
    const int tile = wave * RG + t;   // 8 rows x 4 columns
    const int oh = oh0 + tile % RG * 8 + (px >> 2), ow = ow0 + tile / RG * 4 + (px & 3);
    const bool live = oh < p.out_lo + p.R && ow < p.W_out;
    const size_t yoff = ((size_t)(n * p.y_rows + oh - p.y_row0) * p.W_out + ow) * kMbC;
    const size_t roff = RES ? ((size_t)(n * p.r_rows + oh - p.r_row0) * p.W_out + ow) * kMbC : 0;
    u32x2 o[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int co = g * 8 + kg * 4;
      float v[4] = {acc[t][g * 4 + 0], acc[t][g * 4 + 1], acc[t][g * 4 + 2], acc[t][g * 4 + 3]};
      if (p.bp) {
        const float4 b4 = *(const float4*)(p.bp + co);
        v[0] += b4.x; v[1] += b4.y; v[2] += b4.z; v[3] += b4.w;
      }
      if (RES && live) {
        float r[4];
        unpack4(*(const u32x2*)(p.res + roff + co), r);
        v[0] += r[0]; v[1] += r[1]; v[2] += r[2]; v[3] += r[3];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = clamp_act(v[k], p.cp);
      o[g] = pack4(v);
    }
#pragma unroll
    for (int g = 0; g < 4; g += 2) {
      const auto s0 = __builtin_amdgcn_permlane32_swap(o[g].x, o[g + 1].x, false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(o[g].y, o[g + 1].y, false, false);
      if (live) *(u32x4*)(p.y + yoff + g * 8 + kg * 8) = u32x4{(unsigned)s0[0], (unsigned)s1[0], (unsigned)s0[1], (unsigned)s1[1]};
    }
  }
}

template <int S, bool RES, int ROWS>
__global__ __launch_bounds__(256, S == 1 && ROWS == 8 ? 4 : 3) void mbconv_kernel(const MbParams p) {
  mbconv_body<S, RES, ROWS>(p, blockIdx.x);
}
// The same for several bands of one block in one grid (band b owns blocks first[b] .. first[b + 1]).
template <int S, bool RES, int ROWS>
__global__ __launch_bounds__(256, S == 1 && ROWS == 8 ? 4 : 3) void mbconv_kernel_bands(const Batch<MbParams> t) {
  const int b = batch_find(t, blockIdx.x);
  mbconv_body<S, RES, ROWS>(t.p[b], blockIdx.x - t.first[b]);
}

bool is_pointwise(const OpLaunch& L) {
  return L.op == LOP_CONV2D && L.kh == 1 && L.kw == 1 && L.sh == 1 && L.sw == 1 && L.ph == 0 &&
         L.pw == 0;
}

}  // namespace

// The depthwise weights w[tap][C] (values of the storage type) of a 3 x 3 operator with stride s as
// operands of the 4 x 4 x 4 products: [C / 32][half of the slots][filter row a][quad g of input columns][64
// lanes] x 4 bf16. A lane (block of lanes = channel, lane % 4 = output column m) holds the weights of
// input columns 4 g + {0..3}, i.e. w[a][4 g + k - s m] where that is a tap and zero elsewhere.
size_t mbconv_bands_bytes(int c, int s) { return (size_t)(c / 16) * 3 * (s == 1 ? 2 : 3) * 64 * 8; }
void mbconv_pack_bands(const float* w, int c, int s, unsigned short* dst) {
  const int ks = s == 1 ? 2 : 3;
  for (int cb = 0; cb < c / 16; ++cb)
    for (int a = 0; a < 3; ++a)
      for (int g = 0; g < ks; ++g)
        for (int lane = 0; lane < 64; ++lane)
          for (int k = 0; k < 4; ++k) {
            const int tap = 4 * g + k - s * (lane % 4);
            const int ch = cb / 2 * 32 + slot_channel(dw_slot(lane / 4, cb % 2));
            unsigned bits = 0;
            if (tap >= 0 && tap < 3) memcpy(&bits, &w[(size_t)(a * 3 + tap) * c + ch], 4);
            *dst++ = (unsigned short)(bits >> 16);
          }
}

// Whether the three operators (expand, depthwise, project; shapes and parameters only, the
// slabs are not looked at) can run as one mbconv_kernel launch.
bool mbconv_applies(const OpLaunch& e, const OpLaunch& d, const OpLaunch& p) {
  if (e.dtype != LOP_BF16 || !is_pointwise(e) || !is_pointwise(p)) return false;
  if (e.x.c != kMbC || p.y.c != kMbC || !e.wd16) return false;
  if (e.y.c % 32 != 0 || e.y.c > kMbMaxMid || e.y.c != d.x.c || d.x.c != p.x.c) return false;
  if (d.op != LOP_DWCONV2D || d.kh != 3 || d.kw != 3 || d.ph != 1 || d.pw != 1 || d.dh != 1 ||
      d.dw != 1 || d.sh != d.sw || (d.sh != 1 && d.sh != 2))
    return false;
  return e.res.ptr == nullptr && d.res.ptr == nullptr;
}

// Rows of a workgroup's tile: 16 (stride 1) where that does less work - such a tile costs 1.75 of an 8-row one, having
// a smaller halo, no idle wavefront in the expand part and half the weights to read per pixel - and leaves two
// workgroups per compute unit, 8 otherwise.
static int mb_rows(const OpLaunch& d, const OpLaunch* ps, int n) {
  if (d.sh != 1) return 8;
  long tiles16 = 0, tiles8 = 0;
  for (int b = 0; b < n; ++b) {
    const int R = ps[b].out_hi - ps[b].out_lo;
    if (R <= 0) continue;
    const long row = (long)((ps[b].y.w + 15) / 16) * ps[b].x.n;
    tiles16 += (R + 15) / 16 * row;
    tiles8 += (R + 7) / 8 * row;
  }
  return tiles16 >= 512 && 7 * tiles16 < 4 * tiles8 ? 16 : 8;
}

int mbconv_describe(const OpLaunch& d, const OpLaunch& p, char* name, size_t size) {
  if (name && size)
    snprintf(name, size, "mbconv_kernel<%d, %s, %d>", d.sh, p.res.ptr ? "true" : "false", mb_rows(d, &p, 1));
  return 1;
}

namespace {
MbParams make_mbconv(const OpLaunch& e, const OpLaunch& d, const OpLaunch& p, int th) {
  MbParams q;
  q.x = (const __bf16*)e.x.ptr; q.y = (__bf16*)p.y.ptr; q.res = (const __bf16*)p.res.ptr;
  q.we = e.wd16; q.be = e.bias;
  q.bands = (const float*)d.w + 9 * d.x.c; q.bd = d.bias;
  q.wp = p.wd; q.bp = p.bias;
  q.e_steps = e.k_pad / 32;
  q.x_row0 = e.x.row0; q.x_rows = e.x.rows; q.H = e.x.h; q.W = e.x.w;
  q.y_row0 = p.y.row0; q.y_rows = p.y.rows; q.W_out = p.y.w;
  q.r_row0 = p.res.row0; q.r_rows = p.res.rows;
  q.C_mid = e.y.c; q.nch = e.y.c / 32;
  q.ce = make_clamp(e.act); q.cd = make_clamp(d.act); q.cp = make_clamp(p.act);
  q.out_lo = p.out_lo; q.R = p.out_hi - p.out_lo; q.N = e.x.n;
  const int tw = MbTile<1, 8>::TW;
  q.tiles_x = (q.W_out + tw - 1) / tw;
  q.tiles_y = (q.R + th - 1) / th;
  q.by_tx = make_fastdiv(q.tiles_x); q.by_ty = make_fastdiv(q.tiles_y);
  return q;
}
static_assert(sizeof(Batch<MbParams>) <= 4096, "the parameters of all bands of a launch travel as kernel arguments");
}  // namespace

// Per band: es[b].x the block's input slab; ps[b].y its output slab; ps[b].res residual slab or none;
// ps[b].out_lo/out_hi the output rows to produce.
hipError_t launch_mbconv_bands(const OpLaunch* es, const OpLaunch& d, const OpLaunch* ps, int n, hipStream_t stream,
                               KernelEvents* ev) {
  if (n < 1 || n > kMaxBatch) return hipErrorInvalidValue;
  MbParams qs[kMaxBatch];
  unsigned gx[kMaxBatch];
  int m = 0;
  const int rows = mb_rows(d, ps, n);
  for (int b = 0; b < n; ++b) {
    if (!mbconv_applies(es[b], d, ps[b])) return hipErrorInvalidValue;
    qs[m] = make_mbconv(es[b], d, ps[b], rows);
    if (qs[m].R <= 0 || qs[m].N <= 0) continue;
    gx[m] = (unsigned)(qs[m].tiles_x * qs[m].tiles_y * qs[m].N);
    ++m;
  }
  if (m == 0) return hipSuccess;
  const dim3 block(256);
  if (d.sh == 2)
    return qs[0].res ? launch_group(mbconv_kernel<2, true, 8>, mbconv_kernel_bands<2, true, 8>, qs, m, gx, 1, 1, block, stream, ev)
                     : launch_group(mbconv_kernel<2, false, 8>, mbconv_kernel_bands<2, false, 8>, qs, m, gx, 1, 1, block, stream, ev);
  if (rows == 16)
    return qs[0].res ? launch_group(mbconv_kernel<1, true, 16>, mbconv_kernel_bands<1, true, 16>, qs, m, gx, 1, 1, block, stream, ev)
                     : launch_group(mbconv_kernel<1, false, 16>, mbconv_kernel_bands<1, false, 16>, qs, m, gx, 1, 1, block, stream, ev);
  return qs[0].res ? launch_group(mbconv_kernel<1, true, 8>, mbconv_kernel_bands<1, true, 8>, qs, m, gx, 1, 1, block, stream, ev)
                   : launch_group(mbconv_kernel<1, false, 8>, mbconv_kernel_bands<1, false, 8>, qs, m, gx, 1, 1, block, stream, ev);
}

}  // namespace lop
