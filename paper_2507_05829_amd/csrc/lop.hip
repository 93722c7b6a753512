// C ABI of the library: plan construction (host planning + weight upload), the per-band
// scheduler (compute stream + copy stream + one event per band) and the queries.
#include <hip/hip_runtime.h>

#include <cstdint>

#include <algorithm>
#include <climits>
#include <chrono>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "devmem.hpp"
#include "kernels.hpp"
#include "lop.h"
#include "plan_state.hpp"
#include "plan_tables.hpp"

namespace lop {
hipError_t launch_conv_igemm(const OpLaunch& L, hipStream_t stream, KernelEvents* ev);
hipError_t launch_rowwise_op(const OpLaunch& L, hipStream_t stream, KernelEvents* ev);
hipError_t launch_copy_rows(void* dst, const void* src, size_t pitch, size_t len, int n,
                            hipStream_t stream, int workgroups);
hipError_t launch_fill_words(void* dst, size_t bytes, unsigned word, hipStream_t stream);

hipError_t launch_pointwise(const OpLaunch* Ls, int n, hipStream_t stream, KernelEvents* ev);
size_t mbconv_bands_bytes(int c, int s);
void mbconv_pack_bands(const float* w, int c, int s, unsigned short* dst);
bool mbconv_applies(const OpLaunch& e, const OpLaunch& d, const OpLaunch& p);
int mbconv_describe(const OpLaunch& d, const OpLaunch& p, char* name, size_t size);
hipError_t launch_mbconv_bands(const OpLaunch* es, const OpLaunch& d, const OpLaunch* ps, int n, hipStream_t stream,
                               KernelEvents* ev);
int pointwise_describe(const OpLaunch* Ls, int n, char* name, size_t size);
int conv_igemm_describe(const OpLaunch& L, char* name, size_t size);
int rowwise_describe(const OpLaunch& L, char* name, size_t size);
hipError_t launch_conv_igemm_bands(const OpLaunch* Ls, int n, hipStream_t stream, KernelEvents* ev);
int conv_igemm_describe_bands(const OpLaunch* Ls, int n, char* name, size_t size);
hipError_t launch_rowwise_bands(const OpLaunch* Ls, int n, hipStream_t stream, KernelEvents* ev);
bool dw3_takes(const OpLaunch& L);
hipError_t launch_stem_bands(const OpLaunch* Ls, int n, hipStream_t stream, KernelEvents* ev);

hipError_t launch_op(const OpLaunch& L, hipStream_t stream, KernelEvents* ev) {
  if (L.out_hi <= L.out_lo) return hipSuccess;
  if (L.op == LOP_CONV2D) {
    if (stem_applies(L)) return launch_stem(L, stream, ev);
    return pointwise_applies(L) ? launch_pointwise(&L, 1, stream, ev) : launch_conv_igemm(L, stream, ev);
  }
  return launch_rowwise_op(L, stream, ev);
}

bool stores_second_output(const OpLaunch& L) {
  return L.op != LOP_CONV2D || stem_applies(L) || !pointwise_applies(L);
}

bool op_streams(const OpLaunch& L) {
  return L.op == LOP_CONV2D ? !stem_applies(L) && pointwise_applies(L) : dw3_takes(L);
}

hipError_t launch_op_bands(const OpLaunch* Ls, int n, hipStream_t stream, KernelEvents* ev) {
  if (n < 1 || n > kMaxBandsPerLaunch) return hipErrorInvalidValue;
  if (n == 1) return launch_op(Ls[0], stream, ev);
  if (Ls[0].op == LOP_CONV2D) {
    if (stem_applies(Ls[0])) return launch_stem_bands(Ls, n, stream, ev);
    return pointwise_applies(Ls[0]) ? launch_pointwise(Ls, n, stream, ev) : launch_conv_igemm_bands(Ls, n, stream, ev);
  }
  return launch_rowwise_bands(Ls, n, stream, ev);
}

int describe_op_bands(const OpLaunch* Ls, int n, char* name, size_t size) {
  if (n > 1 && Ls[0].op == LOP_CONV2D && stem_applies(Ls[0])) return stem_describe_bands(Ls, n, name, size);
  if (n > 1 && Ls[0].op == LOP_CONV2D && pointwise_applies(Ls[0])) return pointwise_describe(Ls, n, name, size);
  if (n == 1 || Ls[0].op != LOP_CONV2D) {
    const int k = describe_op(Ls[0], name, size);
    if (n > 1 && name && size) {   // the form that takes several bands carries _bands in its name
      std::string s(name);
      const size_t at = s.find('<');
      s.insert(at == std::string::npos ? s.size() : at, "_bands");
      snprintf(name, size, "%s", s.c_str());
    }
    return k;
  }
  return conv_igemm_describe_bands(Ls, n, name, size);
}

int describe_op(const OpLaunch& L, char* name, size_t size) {
  if (L.op != LOP_CONV2D) return rowwise_describe(L, name, size);
  if (stem_applies(L)) return stem_describe(L, name, size);
  return pointwise_applies(L) ? pointwise_describe(&L, 1, name, size) : conv_igemm_describe(L, name, size);
}
}  // namespace lop

// Scratch of lop_run_chain_static: the slabs of one band at a time and the split-K partial sums
// of one launch at a time, in an array that is part of the loaded code object instead of an
// allocation. Every GPU the library runs on holds its own copy, at its own address, until the
// process ends. In host code this name is only a handle for hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[LOP_STATIC_SCRATCH_BYTES];

namespace {
thread_local int g_last_hip = 0;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each device, once known

// Looks up the address of `scratch` on `device`, which must be the current device. Called when
// a plan is set up on a device, so that lop_run_chain_static itself makes no runtime query.
hipError_t resolve_static_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!ptr) return hipErrorInvalidSymbol;
  g_scratch_ptr[device] = ptr;
  return hipSuccess;
}

void* static_scratch_of(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[device];
}
}  // namespace

namespace lop {
int hip_fail(hipError_t e) {
  g_last_hip = (int)e;
  return e == hipErrorOutOfMemory ? LOP_ERR_OOM : LOP_ERR_HIP;
}
}  // namespace lop

namespace {
using lop::hip_fail;

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

namespace {

int upload_weights(lop_plan_t* P) {
  const lop::Tables& t = P->t;
  const int nl = t.n_layers();
  const bool bf = t.in.dtype == LOP_BF16;
  P->d_w.assign(nl, nullptr);
  P->d_wd.assign(nl, nullptr);
  P->d_wd16.assign(nl, nullptr);
  P->d_w3.assign(nl, nullptr);
  P->d_wstem.assign(nl, nullptr);
  P->d_bias.assign(nl, nullptr);
  for (int l = 0; l < nl; ++l) {
    const lop::LayerInfo& L = t.layers[l];
    const lop_layer_t& d = L.d;
    if (d.op == LOP_CONV2D) {
      if (!d.weight) return LOP_ERR_INVALID_ARG;
      const int kp = P->k_pad[l];
      const int cp = lop::conv_cout_pad(d.c_out);
      const size_t esz = t.esz();
      std::vector<unsigned char> host((size_t)cp * kp * esz, 0);
      // OIHW -> [co][ (a*kw + b)*c_in + ci ]
      for (int co = 0; co < d.c_out; ++co)
        for (int ci = 0; ci < d.c_in; ++ci)
          for (int a = 0; a < d.kh; ++a)
            for (int b = 0; b < d.kw; ++b) {
              const size_t src = (((size_t)co * d.c_in + ci) * d.kh + a) * d.kw + b;
              const size_t dst = (size_t)co * kp + (size_t)(a * d.kw + b) * d.c_in + ci;
              std::memcpy(&host[dst * esz], (const unsigned char*)d.weight + src * esz, esz);
            }
      LOP_HIP(lop::dev_alloc(&P->d_w[l], host.size()));
      LOP_HIP(hipMemcpy(P->d_w[l], host.data(), host.size(), hipMemcpyHostToDevice));
      if (P->has_wstem[l]) {
        // fp32 [c_out / 4][k][4] and, behind it, [c_out / 16][k][16], k = (a*kw + b)*c_in + ci:
        // four (sixteen) weights of one reduction element lie together at an address a whole
        // wavefront shares
        const size_t K = (size_t)d.c_in * d.kh * d.kw;
        std::vector<float> q(2 * (size_t)d.c_out * K);
        for (int co = 0; co < d.c_out; ++co)
          for (size_t k = 0; k < K; ++k) {
            float v;
            const unsigned char* src = &host[((size_t)co * kp + k) * esz];
            if (bf) {
              unsigned short h;
              std::memcpy(&h, src, 2);
              const unsigned u = (unsigned)h << 16;
              std::memcpy(&v, &u, 4);
            } else {
              std::memcpy(&v, src, 4);
            }
            q[((size_t)(co / 4) * K + k) * 4 + co % 4] = v;
            q[(size_t)d.c_out * K + ((size_t)(co / 16) * K + k) * 16 + co % 16] = v;
          }
        if (lop::stem_mfma_shape(d.c_in, d.c_out, d.kh, d.kw)) {   // ... and in the order of the matrix cores
          const size_t at = q.size();
          q.resize(at + lop::stem_mfma_bytes(d.c_out, d.kh, t.in.dtype) / 4, 0.f);
          lop::stem_mfma_pack(host.data(), kp, d.c_out, d.kh, t.in.dtype, (unsigned char*)(q.data() + at));
        }
        LOP_HIP(lop::dev_alloc(&P->d_wstem[l], q.size() * 4));
        LOP_HIP(hipMemcpy(P->d_wstem[l], q.data(), q.size() * 4, hipMemcpyHostToDevice));
      }
      const int ke = 16 / (int)esz;
      if (P->has_wd[l]) {
        // the same values in MFMA operand order: [co / 32][step][half*32 + co % 32] x 16 B
        std::vector<unsigned char> ord(host.size());
        const size_t steps = (size_t)kp / (2 * ke);
        for (int co = 0; co < cp; ++co)
          for (size_t st = 0; st < steps; ++st)
            for (int half = 0; half < 2; ++half) {
              const size_t src = (size_t)co * kp + st * 2 * ke + (size_t)half * ke;
              const size_t dst = (((size_t)(co / 32) * steps + st) * 64 + half * 32 + co % 32) * ke;
              std::memcpy(&ord[dst * esz], &host[src * esz], 16);
            }
        // (fp32 layers: and behind them as three bf16 parts)
        LOP_HIP(lop::dev_alloc(&P->d_wd[l], ord.size() + (P->has_w3[l] ? (size_t)cp * kp * 6 : 0)));
        LOP_HIP(hipMemcpy(P->d_wd[l], ord.data(), ord.size(), hipMemcpyHostToDevice));
        if (P->has_w3[l]) {
          P->d_w3[l] = (char*)P->d_wd[l] + ord.size();
          LOP_HIP(lop::launch_split_weights(P->d_w[l], cp, kp, P->d_w3[l], nullptr));
        }
        if (P->has_wd16[l]) {
          // ... and in the order of 16 x 16 tiles: [co / 16][step][quarter*16 + co % 16] x 16 B
          const size_t steps16 = (size_t)kp / (4 * ke);
          for (int co = 0; co < cp; ++co)
            for (size_t st = 0; st < steps16; ++st)
              for (int q = 0; q < 4; ++q) {
                const size_t src = (size_t)co * kp + st * 4 * ke + (size_t)q * ke;
                const size_t dst = (((size_t)(co / 16) * steps16 + st) * 64 + q * 16 + co % 16) * ke;
                std::memcpy(&ord[dst * esz], &host[src * esz], 16);
              }
          LOP_HIP(lop::dev_alloc(&P->d_wd16[l], ord.size()));
          LOP_HIP(hipMemcpy(P->d_wd16[l], ord.data(), ord.size(), hipMemcpyHostToDevice));
        }
      }
    } else if (d.op == LOP_DWCONV2D) {
      if (!d.weight) return LOP_ERR_INVALID_ARG;
      // C x 1 x kh x kw (storage type) -> [tap][C] fp32
      std::vector<float> host((size_t)d.kh * d.kw * d.c_in);
      for (int c = 0; c < d.c_in; ++c)
        for (int tap = 0; tap < d.kh * d.kw; ++tap) {
          const size_t src = (size_t)c * d.kh * d.kw + tap;
          float v;
          if (bf) {
            const unsigned u = (unsigned)((const unsigned short*)d.weight)[src] << 16;
            std::memcpy(&v, &u, 4);
          } else {
            v = ((const float*)d.weight)[src];
          }
          host[(size_t)tap * d.c_in + c] = v;
        }
      if (bf && d.c_in % 32 == 0 && d.kh == 3 && d.kw == 3 && d.sh == d.sw && (d.sh == 1 || d.sh == 2)) {
        // ... and behind it the same weights as the fused block kernel's matrix operands
        const size_t at = host.size();
        host.resize(at + lop::mbconv_bands_bytes(d.c_in, d.sh) / 4);
        lop::mbconv_pack_bands(host.data(), d.c_in, d.sh, (unsigned short*)(host.data() + at));
      }
      LOP_HIP(lop::dev_alloc(&P->d_w[l], host.size() * 4));
      LOP_HIP(hipMemcpy(P->d_w[l], host.data(), host.size() * 4, hipMemcpyHostToDevice));
    }
    if (d.bias && d.op != LOP_MAXPOOL2D) {
      LOP_HIP(lop::dev_alloc((void**)&P->d_bias[l], (size_t)d.c_out * 4));
      LOP_HIP(hipMemcpy(P->d_bias[l], d.bias, (size_t)d.c_out * 4, hipMemcpyHostToDevice));
    }
  }
  return LOP_OK;
}

// The images a merged chain's launches work on while it is enqueued: they lie from image `first` on
// in the caller's tensors, and from the buffers' beginning in the arena. rows: the pass's rows, where
// those are a part of the chain's.
struct ChainPass {
  lop_plan_t* P;
  ChainPass(lop_plan_t* plan, int first, int images, lop_rows_t rows = {0, 0}) : P(plan) {
    P->pass_first = first; P->pass_images = images; P->pass_rows = rows;
  }
  ~ChainPass() { P->pass_first = 0; P->pass_images = 0; P->pass_rows = {0, 0}; }
};

// Last launch (by the index of the layer it ends with) that reads layer l's output, under either
// set of fused groups; l itself if nobody does.
int last_reader(const lop_plan_t* P, int l) {
  const lop::Tables& t = P->t;
  const int nl = t.n_layers();
  int last = l;
  for (int j = l + 1; j < nl; ++j) {
    if (t.layers[j].d.input_from != l && t.layers[j].d.residual_from != l) continue;
    last = std::max(last, j);
    for (const Fusion* F : {&P->fuse_band, &P->fuse_chain})
      for (int q = j; q < nl; ++q)   // (a layer inside a group is read when the group's last layer runs)
        if (F->head[q] >= 0 && F->head[q] <= j) last = std::max(last, q);
  }
  return last;
}

// Offsets for the layers' outputs in one arena: a buffer is live from its layer's launch to its
// last reader's, and layers whose buffers are never live together share memory, so that what a
// chain keeps between launches is a few layers' rows instead of all of them (the rows stay in
// the caches, and a quarter of the memory holds a whole chain). size[l] == 0: no buffer.
size_t place_slabs(const lop_plan_t* P, const std::vector<size_t>& size, std::vector<size_t>* off) {
  const int nl = P->t.n_layers();
  std::vector<int> last(nl);
  for (int l = 0; l < nl; ++l) last[l] = last_reader(P, l);
  size_t worst = 0;
  for (int l = 0; l + 1 < nl; ++l) {  // the last layer writes the caller's output
    (*off)[l] = 0;
    if (!size[l]) continue;
    size_t at = 0;
    for (bool moved = true; moved;) {   // the lowest place that touches no buffer still live
      moved = false;
      for (int k = 0; k < l; ++k)
        if (size[k] && last[k] >= l && at < (*off)[k] + size[k] && (*off)[k] < at + size[l]) {
          at = (*off)[k] + size[k];
          moved = true;
        }
    }
    (*off)[l] = at;
    worst = std::max(worst, at + size[l]);
  }
  return worst;
}

// Whether every layer's output row depends on that row of its input only (chains of row-wise operators).
bool keeps_to_rows(const lop_plan_t* P) {
  for (const lop::LayerInfo& L : P->t.layers)
    if (L.d.op == LOP_MAXPOOL2D || L.d.kh != 1 || L.d.sh != 1 || L.d.ph != 0) return false;
  return true;
}
// The result rows of bands [first, last).
lop_rows_t pass_rows(const lop_plan_t* P, int first, int last) {
  lop_rows_t r = {0, 0};
  for (int b = first; b < last; ++b) {
    const lop_rows_t q = P->t.bands[b].need[P->t.n_layers()];
    if (q.hi <= q.lo) continue;
    r = r.hi <= r.lo ? q : lop_rows_t{std::min(r.lo, q.lo), std::max(r.hi, q.hi)};
  }
  return r;
}

lop::OpLaunch make_launch(const lop_plan_t* P, int band, int l, const void* d_in, void* d_out);

// Split-K workspace of the launch that computes layer l (a dense convolution of its own) for these bands.
size_t group_workspace(const std::vector<lop::OpLaunch>& group) {
  if (group.empty() || lop::pointwise_applies(group[0])) return 0;
  return lop::conv_workspace_bytes_bands(group.data(), (int)group.size());
}
bool launches_alone(const lop_plan_t* P, const Fusion& F, int l) {
  return P->t.layers[l].d.op == LOP_CONV2D && !F.away[l] && F.head[l] < 0;
}

// Largest split-K workspace of the launches that compute one band (the launch descriptors only
// need sizes here, not the scratch addresses).
size_t band_workspace(const lop_plan_t* P) {
  size_t most = 0;
  for (int l = 0; l < P->t.n_layers(); ++l) {
    if (!launches_alone(P, P->fuse_band, l) && !(P->batched && launches_alone(P, P->fuse_chain, l))) continue;
    for (int b = 0; b < P->t.n_bands; ++b) {
      const lop_rows_t r = P->t.bands[b].compute[l];
      if (r.hi > r.lo) most = std::max(most, group_workspace({make_launch(P, b, l, nullptr, nullptr)}));
    }
  }
  return most;
}

// ... and of the launches of a merged chain (kGrouped, kWhole), over the passes that enqueue_merged_kernels
// makes. A last pass over fewer images is looked at by itself: fewer pixels can mean more slices, or a kernel
// that cuts the reduction where the larger launch has one that does not.
size_t merged_workspace(lop_plan_t* P) {
  const int nb = P->t.n_bands, nl = P->t.n_layers(), rest = P->t.in.n % P->images;
  size_t most = 0;
  auto pass = [&](int images, int first, int last, int layer, int layers) {
    const bool whole = P->sched == ChainSched::kWhole;
    const lop_rows_t rows = whole && P->group < nb ? pass_rows(P, first, last) : lop_rows_t{0, 0};
    if (whole && P->group < nb && rows.hi <= rows.lo) return;
    const ChainPass sized(P, 0, images, rows);
    std::vector<lop::OpLaunch> group;
    for (int l = layer; l < layers; ++l) {
      if (!launches_alone(P, P->fuse_chain, l)) continue;
      if (whole) {
        most = std::max(most, group_workspace({make_launch(P, P->t.whole(), l, nullptr, nullptr)}));
        continue;
      }
      for (int b = first; b < last; b += lop::kMaxBandsPerLaunch) {   // (a launch keeps all its bands' partial sums at once)
        group.clear();
        for (int k = b; k < std::min(last, b + lop::kMaxBandsPerLaunch); ++k)
          if (P->t.bands[k].compute[l].hi > P->t.bands[k].compute[l].lo) group.push_back(make_launch(P, k, l, nullptr, nullptr));
        most = std::max(most, group_workspace(group));
      }
    }
  };
  const int in_passes = P->cut < 0 ? nl : P->cut + 1;
  for (int b = 0; b < nb; b += P->group) {
    pass(P->images, b, std::min(nb, b + P->group), 0, in_passes);
    if (rest) pass(rest, b, std::min(nb, b + P->group), 0, in_passes);
  }
  if (in_passes < nl) pass(P->t.in.n, 0, nb, in_passes, nl);
  return most;
}

// The scratch of a merged chain (kGrouped, kWhole), what it keeps between launches and the largest workspace
// of a launch, fits this: images of a batch, and then bands, are dealt to passes of equal size, as few as
// do. It is the size of the static array, so that lop_run_chain_static, which has no more than that, runs
// the launches lop_run_chain does and takes every plan whose bands fit there one by one;
// and it is a quarter of the 256 MB Infinity Cache, so that four chains in flight keep their
// intermediate rows on the chip. A chain too large even for one image (or one band of one image)
// runs band by band: its launches are long enough by themselves.
constexpr size_t kMergeMaxBytes = LOP_STATIC_SCRATCH_BYTES;
constexpr size_t kLaneSlabsMax = (size_t)192 << 20;
// A chain of row-wise operators has no halo, and callers that stream matrix rows run its bands one
// by one: a chain of few rows and few products (rows x columns in x columns out of its largest layer) runs the bands' own
// launches, so that its results are those of lop_run_band bit for bit, as lop.h says. That is the only reason: merged it
// is faster at every size (us a call with calls in flight and alone, four bands band by band -> merged: bf16 256 rows x 256 -> 1024 -> 256
// 24.8, 57 -> 8.3, 22; 1 000 x 256 -> 256 -> 256 25.6, 57 -> 8.3, 19; 2 000 x 128 -> 256 -> 128 25.4, 56 -> 8.0, 19; fp32 1 000 x 256 ->
// 256 -> 256 25.6, 59 -> 7.6, 22), so chains of many rows merge whatever their products (3 000 x 128 -> 256 -> 128 in eight bands 48, 80
// -> 8.1, 21) and those of many products whatever their rows (256 x 1024 -> 4096 -> 1024 61 -> 20).
constexpr int kMergeMinRows = 2048;
constexpr size_t kMergeMinProducts = (size_t)1 << 27;

void size_scratch(lop_plan_t* P) {
  const lop::Tables& t = P->t;
  const int nl = t.n_layers(), nb = t.n_bands, n = t.in.n;
  // (a buffer in the bands' own slabs, and one of a merged chain, for the layers that store their rows there; the
  // measurement aids of a plan with batched launches run those layer by layer on the bands' slabs)
  auto band_keeps = [&](int l) { return !P->fuse_band.away[l] || (P->batched && !P->fuse_chain.away[l]); };
  auto chain_keeps = [&](int l) { return !P->fuse_chain.away[l]; };
  auto rows_bytes = [&](int images, int l, int rows) {
    return rows > 0 ? align_up((size_t)images * rows * t.row_elems(l) * t.esz(), 256) : (size_t)0;
  };
  auto band_rows = [&](int b, int l) { return t.bands[b].need[l + 1].hi - t.bands[b].need[l + 1].lo; };
  std::vector<size_t> size(nl, 0);
  // buffers of a whole chain, of at most `rows` rows
  auto place_whole = [&](int images, int rows) {
    for (int l = 0; l + 1 < nl; ++l) size[l] = chain_keeps(l) ? rows_bytes(images, l, std::min(rows, t.layers[l].h_out)) : 0;
    return place_slabs(P, size, &P->chain_off[nb]);
  };
  // the slabs of bands [b0, b1) at once: one block per layer, the bands' slabs one behind the other in it
  auto place_bands = [&](int images, int b0, int b1, auto keeps, std::vector<std::vector<size_t>>* off) {
    for (int l = 0; l + 1 < nl; ++l) {
      size[l] = 0;
      for (int b = b0; b < b1 && keeps(l); ++b) size[l] += rows_bytes(images, l, band_rows(b, l));
    }
    std::vector<size_t> block(nl, 0);
    const size_t bytes = place_slabs(P, size, &block);
    for (int l = 0; l + 1 < nl; ++l) {
      size_t at = block[l];
      for (int b = b0; b < b1 && keeps(l); ++b) {
        (*off)[b][l] = at;
        at += rows_bytes(images, l, band_rows(b, l));
      }
    }
    return bytes;
  };
  auto place_groups = [&](int images, int per, auto keeps, std::vector<std::vector<size_t>>* off) {
    size_t most = 0;
    for (int b = 0; b < nb; b += per) most = std::max(most, place_bands(images, b, std::min(nb, b + per), keeps, off));
    return most;
  };

  // A chain whose passes end with layer c: that layer's rows of all images and bands in front (kept bytes), behind them what a
  // pass of `images` images and `per` bands keeps of the layers before it, or (all images and bands) what the layers behind
  // it keep.
  size_t kept = 0;
  auto place_cut = [&](int c, int images, int per, bool whole) {
    const bool behind = images == n && per == nb;
    size_t most = 0;
    kept = 0;
    if (whole) {
      P->chain_off[nb][c] = 0;
      kept = rows_bytes(n, c, t.layers[c].h_out);
    } else {
      for (int b = 0; b < nb; ++b) {
        P->chain_off[b][c] = kept;
        kept += rows_bytes(n, c, band_rows(b, c));
      }
    }
    auto place = [&](int b0, int b1) {
      for (int l = 0; l + 1 < nl; ++l) {
        size[l] = 0;
        if (l == c ? !behind : behind != (l > c) || !chain_keeps(l)) continue;
        if (l == c) size[l] = kept;
        else if (whole) size[l] = rows_bytes(images, l, t.layers[l].h_out);
        else for (int b = b0; b < b1; ++b) size[l] += rows_bytes(images, l, band_rows(b, l));
      }
      std::vector<size_t> block(nl, 0);
      const size_t bytes = place_slabs(P, size, &block);
      for (int l = 0; l + 1 < nl; ++l) {
        if (l == c || !size[l]) continue;
        size_t at = block[l] + (behind ? 0 : kept);
        if (whole) { P->chain_off[nb][l] = at; continue; }
        for (int b = b0; b < b1; ++b) {
          P->chain_off[b][l] = at;
          at += rows_bytes(images, l, band_rows(b, l));
        }
      }
      most = std::max(most, bytes + (behind ? 0 : kept));
    };
    for (int b = 0; b < nb; b += per) place(b, std::min(nb, b + per));
    return most;
  };

  // bands that run one by one: in reuse mode on one full-height buffer per layer (rows at their
  // absolute position), kept from band to band
  P->sched = ChainSched::kPerBand;
  P->group = nb;
  P->images = n;
  P->cut = -1;
  P->cut_bytes = 0;
  P->slab_off.assign(nb + 1, std::vector<size_t>(nl, 0));   // (descriptors of the whole chain are made outside of a pass, too)
  P->chain_off.assign(nb + 1, std::vector<size_t>(nl, 0));
  P->arena_bytes = 0;
  if (t.reuse) {
    for (int l = 0; l + 1 < nl; ++l) {
      for (int b = 0; b < nb; ++b) P->slab_off[b][l] = P->arena_bytes;
      if (band_keeps(l)) P->arena_bytes += rows_bytes(n, l, t.layers[l].h_out);
    }
  } else {
    P->arena_bytes = place_groups(n, 1, band_keeps, &P->slab_off);
  }
  P->conv_ws_bytes = band_workspace(P);

  // Merged launches in place of them, if they fit: one plan holds one arena and one workspace for both.
  const size_t arena = P->arena_bytes, ws = P->conv_ws_bytes;
  const bool bands_fit = align_up(arena, 256) + ws <= kMergeMaxBytes;
  auto merge = [&](ChainSched sched, int images, int per, size_t merged, bool always) {
    P->sched = sched; P->images = images; P->group = per;
    if (always || merged <= kMergeMaxBytes) {
      const size_t merged_ws = merged_workspace(P), both = std::max(arena, merged), both_ws = std::max(ws, merged_ws);
      if (always || (bands_fit ? align_up(both, 256) + both_ws : align_up(merged, 256) + merged_ws) <= kMergeMaxBytes) {
        P->arena_bytes = both;
        P->conv_ws_bytes = both_ws;
        return true;
      }
    }
    P->sched = ChainSched::kPerBand; P->images = n; P->group = nb;
    return false;
  };
  if (P->batched) {
    merge(ChainSched::kGrouped, n, nb, place_groups(n, nb, chain_keeps, &P->chain_off), true);
    return;
  }
  size_t products = 0;
  for (const lop::LayerInfo& L : t.layers) products = std::max(products, (size_t)n * L.h_out * L.d.c_in * L.d.c_out);
  const bool few_rows = t.in.w == 1 && n * t.in.h < kMergeMinRows && products < kMergeMinProducts;
  if ((P->flags & LOP_FLAG_PLAN_ONLY) || (few_rows && nb > 1)) return;
  const bool whole = t.disjoint();
  // Launches that stream memory (1 x 1 and depthwise layers by themselves) gain from being merged what launches cost, and
  // lose the lanes that would run them side by side: no more passes than a lane has bands. Inverted-residual chains
  // layer by layer, eight bands, us a call band by band -> merged: one image of 400 x 400 (two passes) 312 -> 140, 391 -> 336
  // alone; 640 x 640 (four) 406 -> 325, but 484 -> 713 alone; two of 512 x 512 (eight) 480 -> 457, 567 -> 1 024 alone; eight
  // of 640 x 640 (32) 2.2 -> 3.3 ms.
  bool streams = false;
  for (int l = 0; l < nl; ++l)
    streams = streams || (!P->fuse_chain.away[l] && P->fuse_chain.head[l] < 0 && lop::op_streams(lop::describe_layer(P, l)));
  const int most = streams ? std::max(1, nb / LOP_DEFAULT_LANES) : INT_MAX;
  // Passes only as far as the chain is too large: where some layer's rows of all images and bands fit beside a pass and
  // nothing behind that layer reads what lies in front of it, the layers behind it run once (the fewest launches are taken).
  // A pass of the small layers of a chain's end fills no chip: us a call, all layers in passes -> cut, in flight (alone): detector
  // of 720 x 1280 in 16 bands 148 -> 144 (298 -> 277); VGG-16 stack on two images of 288 x 288 458 -> 438 (678 -> 597);
  // inverted-residual chain on eight images of 640 x 640 571 -> 563 (886 -> 863), reusing rows 412 -> 400.
  struct Cut { int layer, images, per; long launches; };
  auto cuts_of = [&]() {
    std::vector<Cut> cuts;
    auto launches = [&](int lo, int hi) {
      long m = 0;
      for (int l = lo; l < hi; ++l) m += !P->fuse_chain.away[l];
      return m;
    };
    for (int c = 0; c + 1 < nl; ++c) {
      bool ok = !P->fuse_chain.away[c] && (n == 1 || (size_t)t.row_elems(c) * t.esz() % 16 == 0);
      for (int l = c + 1; l < nl && ok; ++l) {
        const lop_layer_t& d = t.layers[l].d;
        ok = d.input_from >= c && (d.residual_from == LOP_NO_RESIDUAL || d.residual_from >= c) && (P->fuse_chain.head[l] < 0 || P->fuse_chain.head[l] > c);
      }
      if (!ok) continue;
      const size_t behind = place_cut(c, n, nb, whole);
      if (behind > kMergeMaxBytes) continue;
      for (int passes = 2; passes <= n + (whole ? 0 : nb - 1); ++passes) {   // images first, then groups of bands
        int images = (n + std::min(passes, n) - 1) / std::min(passes, n), per = nb;
        if (passes > n) { const int groups = passes - n + 1; images = 1; per = (nb + groups - 1) / groups; }
        if (place_cut(c, images, per, whole) > kMergeMaxBytes) continue;
        const long made = (long)((n + images - 1) / images) * ((nb + per - 1) / per);
        if (made <= most) cuts.push_back({c, images, per, made * launches(0, c + 1) + launches(c + 1, nl)});
        break;
      }
    }
    std::sort(cuts.begin(), cuts.end(), [](const Cut& a, const Cut& b) { return a.launches < b.launches; });
    return cuts;
  };
  auto merge_passes = [&]() {
    for (int passes = 1, images = 0; images != 1; ++passes) {
      images = (n + passes - 1) / passes;
      if (!whole && (n + images - 1) / images > most) return false;
      if (whole ? merge(ChainSched::kWhole, images, nb, place_whole(images, INT_MAX), false)
                : merge(ChainSched::kGrouped, images, nb, place_groups(images, nb, chain_keeps, &P->chain_off), false))
        return true;
    }
    for (int groups = 2, per = nb; !whole && per != 1; ++groups) {
      per = (nb + groups - 1) / groups;
      if (n * ((nb + per - 1) / per) > most) return false;
      if (merge(ChainSched::kGrouped, 1, per, place_groups(1, per, chain_keeps, &P->chain_off), false)) return true;
    }
    return false;
  };
  if (merge_passes()) {
    const long passes = (long)((n + P->images - 1) / P->images) * ((nb + P->group - 1) / P->group);
    if (passes == 1) return;
    long layers = 0;
    for (int l = 0; l < nl; ++l) layers += !P->fuse_chain.away[l];
    const ChainSched sched = P->sched;
    const int images = P->images, per = P->group;
    const size_t arena_bytes = P->arena_bytes, ws_bytes = P->conv_ws_bytes;
    const std::vector<std::vector<size_t>> off = P->chain_off;
    for (const Cut& c : cuts_of()) {
      if (c.launches >= passes * layers) break;
      const size_t behind = place_cut(c.layer, n, nb, whole), in_pass = place_cut(c.layer, c.images, c.per, whole);
      P->cut = c.layer;
      P->cut_bytes = kept;
      if (merge(sched, c.images, c.per, std::max(behind, in_pass), false)) return;
    }
    P->cut = -1; P->cut_bytes = 0; P->sched = sched; P->images = images; P->group = per;
    P->arena_bytes = arena_bytes; P->conv_ws_bytes = ws_bytes; P->chain_off = off;
    return;
  }
  // a chain whose layers keep to their rows: passes over the rows of as many bands as fit, if two do (the launches of
  // one band at a time are better off on four lanes: alone 1 150 against 1 390 us on 65 536 x 1024 -> 4096 -> 1024).
  // Band by band the launches leave their last rounds of tiles to compete: 16 425 x 816 -> 2552 -> 816
  // in five bands 271 -> 176 us a chain, 32 768 x 1024 -> 4096 -> 1024 in eight 785 -> 552.
  for (int passes = 2; whole && keeps_to_rows(P); ++passes) {
    const int per = (nb + passes - 1) / passes;
    if (per < 2) return;
    int rows = 0;
    for (int b = 0; b < nb; b += per) { const lop_rows_t r = pass_rows(P, b, std::min(nb, b + per)); rows = std::max(rows, r.hi - r.lo); }
    if (merge(ChainSched::kWhole, 1, per, place_whole(1, rows), false)) return;
  }
}

// Whether LOP_FLAG_BATCH_BANDS is open to the plan: not to inverted-residual blocks and streaming launches, whose callers
// are told so; lop_run_chain merges those where it pays.
bool all_launches_batchable(const lop_plan_t* P) {
  const lop::Tables& t = P->t;
  if (t.n_bands > lop::kMaxBandsPerLaunch) return false;
  for (int l = 0; l < t.n_layers(); ++l) {
    if (P->fuse_chain.away[l]) continue;
    if (P->fuse_chain.head[l] >= 0) {
      if (P->fuse_chain.head[l] != l - 1) return false;   // an inverted-residual block
      continue;
    }
    if (lop::op_streams(lop::describe_layer(P, l))) return false;
  }
  return true;
}

lop::Slab slab_of(const lop_plan_t* P, int band, int tensor, const void* d_in, void* d_out) {
  const lop::Tables& t = P->t;
  const int nl = t.n_layers();
  lop::Slab s;
  s.n = P->pass_images ? P->pass_images : t.in.n;
  s.h = t.tensor_h(tensor);
  auto from_pass = [&](const void* base) -> void* {   // a caller's tensor, from the pass's first image on
    return base ? (char*)const_cast<void*>(base) + (size_t)P->pass_first * s.h * t.row_elems(tensor) * t.esz() : nullptr;
  };
  if (tensor < 0) {
    s.ptr = from_pass(d_in);
    s.w = t.in.w; s.c = t.in.c; s.row0 = 0; s.rows = t.in.h;
  } else {
    s.w = t.layers[tensor].w_out;
    s.c = t.layers[tensor].d.c_out;
    if (tensor == nl - 1) {
      s.ptr = from_pass(d_out); s.row0 = 0; s.rows = s.h;
    } else {
      // (no arena yet while the plan is being sized, and none at all in a plan-only plan)
      char* const arena = (char*)P->arena_of(band);
      s.ptr = arena ? arena + (P->pass_images ? P->chain_off : P->slab_off)[band][tensor] : nullptr;
      if (P->pass_rows.hi > P->pass_rows.lo) {
        s.row0 = P->pass_rows.lo; s.rows = P->pass_rows.hi - P->pass_rows.lo;
      } else if (t.reuse) {
        s.row0 = 0; s.rows = s.h;
      } else {
        const lop_rows_t r = t.bands[band].need[tensor + 1];
        s.row0 = r.lo; s.rows = r.hi - r.lo;
      }
      // (the passes' last layer keeps all images)
      if (P->pass_images && tensor == P->cut && s.ptr) s.ptr = (char*)s.ptr + (size_t)P->pass_first * s.rows * t.row_elems(tensor) * t.esz();
    }
  }
  return s;
}

lop::OpLaunch make_launch(const lop_plan_t* P, int band, int l, const void* d_in, void* d_out) {
  const lop::Tables& t = P->t;
  const lop::LayerInfo& L = t.layers[l];
  lop::OpLaunch o;
  o.op = L.d.op;
  o.dtype = t.in.dtype;
  o.x = slab_of(P, band, L.d.input_from, d_in, d_out);
  o.y = slab_of(P, band, l, d_in, d_out);
  if (L.d.residual_from != LOP_NO_RESIDUAL) o.res = slab_of(P, band, L.d.residual_from, d_in, d_out);
  if (!P->d_w.empty()) {  // uploaded (a plan-only plan has tables but no device arrays)
    o.w = P->d_w[l];
    o.wd = P->d_wd[l];
    o.wd16 = P->d_wd16[l];
    o.w3 = P->d_w3[l];
    o.wstem = P->d_wstem[l];
    o.bias = P->d_bias[l];
  } else {
    // not uploaded (yet): the kernel choice only asks which packings exist, so a marker that
    // is never dereferenced stands for each that upload_weights would make
    o.wd = P->has_wd[l] ? (const void*)P : nullptr;
    o.wd16 = P->has_wd16[l] ? (const void*)P : nullptr;
    o.w3 = P->has_w3[l] ? (const void*)P : nullptr;
    o.wstem = P->has_wstem[l] ? (const void*)P : nullptr;
  }
  o.k_pad = P->k_pad[l];
  o.kh = L.d.kh; o.kw = L.d.kw; o.sh = L.d.sh; o.sw = L.d.sw;
  o.ph = L.d.ph; o.pw = L.d.pw; o.dh = L.d.dh; o.dw = L.d.dw;
  o.act = L.d.act;
  o.alone = P->alone;
  const lop_rows_t rows = P->pass_rows.hi > P->pass_rows.lo ? P->pass_rows : t.bands[band].compute[l];
  o.out_lo = rows.lo;
  o.out_hi = rows.hi;
  o.ws = P->ws_of(band);
  o.ws_bytes = P->conv_ws_bytes;
  return o;
}

}  // namespace

namespace lop {
OpLaunch describe_layer(const lop_plan_s* P, int l) {
  const lop::LayerInfo& L = P->t.layers[l];
  lop::OpLaunch o;
  o.op = L.d.op;
  o.dtype = P->t.in.dtype;
  o.x.c = L.d.c_in; o.y.c = L.d.c_out;
  o.x.n = o.y.n = P->t.in.n;
  if (L.d.residual_from != LOP_NO_RESIDUAL) o.res.ptr = const_cast<lop_plan_t*>(P);
  if (!P->d_w.empty()) {  // uploaded (not a plan-only plan)
    o.w = P->d_w[l]; o.wd = P->d_wd[l]; o.wd16 = P->d_wd16[l]; o.w3 = P->d_w3[l]; o.wstem = P->d_wstem[l]; o.bias = P->d_bias[l];
  } else {
    o.wd = P->has_wd[l] ? (const void*)P : nullptr;
    o.wd16 = P->has_wd16[l] ? (const void*)P : nullptr;
    o.w3 = P->has_w3[l] ? (const void*)P : nullptr;
    o.wstem = P->has_wstem[l] ? (const void*)P : nullptr;
  }
  o.k_pad = P->k_pad[l];
  o.kh = L.d.kh; o.kw = L.d.kw; o.sh = L.d.sh; o.sw = L.d.sw;
  o.ph = L.d.ph; o.pw = L.d.pw; o.dh = L.d.dh; o.dw = L.d.dw;
  o.act = L.d.act;
  return o;
}
}  // namespace lop

namespace {
using lop::describe_layer;

// Groups of three layers that run as one launch (an inverted-residual block): layer h a 1x1
// conv, h + 1 a depthwise conv reading only h, h + 2 a 1x1 conv reading only h + 1, and
// nobody else reads h or h + 1. Then groups of two: a dense conv and the max
// pooling that is its only reader (see convpool_applies), where that pays for launches of one band (merged false) or
// of all bands (merged true).
void find_fused_groups(lop_plan_t* P, bool merged, Fusion* F) {
  const lop::Tables& t = P->t;
  const int nl = t.n_layers();
  F->head.assign(nl, -1);
  F->away.assign(nl, 0);
  if (P->flags & (LOP_FLAG_NO_FUSE | LOP_FLAG_PLAN_ONLY)) return;
  for (int h = 0; h + 2 < nl; ++h) {
    if (F->away[h] || F->head[h] >= 0) continue;
    const int m = h + 1, q = h + 2;
    if (t.layers[m].d.input_from != h || t.layers[q].d.input_from != m) continue;
    bool shared = false;
    for (int j = 0; j < nl; ++j) {
      const lop_layer_t& d = t.layers[j].d;
      if (j != m && d.input_from == h) shared = true;
      if (j != q && d.input_from == m) shared = true;
      if (d.residual_from == h || d.residual_from == m) shared = true;
    }
    if (shared) continue;
    if (!lop::mbconv_applies(describe_layer(P, h), describe_layer(P, m), describe_layer(P, q))) continue;
    F->head[q] = h;
    F->away[h] = F->away[m] = 1;
    h = q;
  }
  // The launch computes the rows of the conv under its pooling windows: those have to be the rows the plan has it
  // compute. (Windows that do not overlap: in every mode. With overlapping ones not where bands share rows.)
  const bool whole = t.disjoint();
  for (int h = 0; h + 1 < nl; ++h) {
    const int q = h + 1;
    if (F->away[h] || F->head[h] >= 0 || F->away[q] || F->head[q] >= 0) continue;
    if (t.layers[q].d.input_from != h) continue;
    bool shared = false;
    for (int j = 0; j < nl; ++j) {
      const lop_layer_t& d = t.layers[j].d;
      if (j != q && d.input_from == h) shared = true;
      if (d.residual_from == h) shared = true;
    }
    if (shared) continue;
    if (!lop::convpool_applies(describe_layer(P, h), describe_layer(P, q))) continue;
    // (a first layer keeps its own launches for bands one by one, whose callers time and watch layer by layer)
    if (!merged && lop::stem_pool_applies(describe_layer(P, h), describe_layer(P, q))) continue;
    const lop::LayerInfo& C = t.layers[h];
    const size_t esz = t.esz();
    if ((size_t)C.n * C.h_in * C.w_in * C.d.c_in * esz >= ((size_t)1 << 31)) continue;  // 32-bit offsets
    bool fits = true;
    std::vector<lop::OpLaunch> convs;
    auto take = [&](int b) {
      const lop_rows_t pr = t.bands[b].compute[q], cr = t.bands[b].compute[h];
      if (pr.hi <= pr.lo) { fits = fits && cr.hi <= cr.lo; return; }
      const lop_layer_t& w = t.layers[q].d;
      fits = fits && cr.lo == std::max(0, pr.lo * w.sh - w.ph) && cr.hi == std::min(C.h_out, (pr.hi - 1) * w.sh - w.ph + w.kh);
      if (fits) convs.push_back(make_launch(P, b, h, nullptr, nullptr));
    };
    if (merged && whole) take(t.whole());
    else for (int b = 0; b < t.n_bands; ++b) take(b);
    if (!fits) continue;
    if (merged) {
      for (size_t at = 0; at < convs.size(); at += lop::kMaxBandsPerLaunch)
        fits = fits && lop::convpool_pays_bands(&convs[at], (int)std::min<size_t>(lop::kMaxBandsPerLaunch, convs.size() - at));
    } else {
      for (const auto& c : convs) fits = fits && lop::convpool_pays_bands(&c, 1);
    }
    if (!fits) continue;
    F->head[q] = h;
    F->away[h] = 1;
  }
}

// The groups of a band's own launches; a plan that asks for batched launches describes those.
const Fusion& band_fusion(const lop_plan_t* P) { return P->batched ? P->fuse_chain : P->fuse_band; }

// Whether layer l ends a conv + pooling group (else, if it ends a group, an inverted-residual block).
bool ends_convpool(const Fusion& F, int l) { return F.head[l] >= 0 && F.head[l] == l - 1; }

// The two descriptors of a conv + pooling launch of one band.
void convpool_launches(const lop_plan_t* P, int band, int l, const void* d_in, void* d_out,
                       lop::OpLaunch* conv, lop::OpLaunch* pool) {
  *pool = make_launch(P, band, l, d_in, d_out);
  *conv = make_launch(P, band, l - 1, d_in, d_out);   // (its y slab is never used: the layer has no buffer)
}

// The first and the last operator of an inverted-residual block's launch of one band: the block's
// input slab, its output slab, residual and rows.
void mbconv_launches(const lop_plan_t* P, int head, int band, int l, const void* d_in, void* d_out, lop::OpLaunch* e,
                     lop::OpLaunch* p) {
  *e = describe_layer(P, head);
  e->x = slab_of(P, band, P->t.layers[head].d.input_from, d_in, d_out);
  *p = make_launch(P, band, l, d_in, d_out);
}

// Rows of layer l one launch of band `band` produces (none for a layer that is part of a
// later layer's launch).
lop_rows_t launch_rows(const lop_plan_t* P, const Fusion& F, int band, int l) {
  if (F.away[l]) return lop_rows_t{0, 0};
  return P->t.bands[band].compute[l];
}

// Enqueue what produces layer l's rows of one band (or, band t.whole(), of the whole chain): its
// own kernel(s), or the fused launch of the group it ends.
hipError_t launch_layer(const lop_plan_t* P, const Fusion& F, int band, int l, const void* d_in, void* d_out,
                        hipStream_t cs, lop::KernelEvents* ev = nullptr, void* y2 = nullptr) {
  const lop_rows_t r = launch_rows(P, F, band, l);
  if (r.hi <= r.lo) return hipSuccess;
  if (F.head[l] < 0) {
    lop::OpLaunch o = make_launch(P, band, l, d_in, d_out);
    o.y2 = y2;
    return lop::launch_op(o, cs, ev);
  }
  if (ends_convpool(F, l)) {
    lop::OpLaunch conv, pool;
    convpool_launches(P, band, l, d_in, d_out, &conv, &pool);
    pool.y2 = y2;
    return lop::launch_convpool(conv, pool, cs, ev);
  }
  lop::OpLaunch e, p;
  mbconv_launches(P, F.head[l], band, l, d_in, d_out, &e, &p);
  return lop::launch_mbconv_bands(&e, describe_layer(P, F.head[l] + 1), &p, 1, cs, ev);
}

// Kernel name (and reduction slices) of that launch.
int describe_layer_launch(const lop_plan_t* P, int band, int l, char* name, size_t size) {
  const Fusion& F = P->fuse_band;
  const lop_rows_t r = launch_rows(P, F, band, l);
  if (r.hi <= r.lo) return 0;
  if (F.head[l] < 0) return lop::describe_op(make_launch(P, band, l, nullptr, nullptr), name, size);
  if (ends_convpool(F, l)) {
    lop::OpLaunch conv, pool;
    convpool_launches(P, band, l, nullptr, nullptr, &conv, &pool);
    return lop::convpool_describe(conv, pool, name, size);
  }
  lop::OpLaunch p = make_launch(P, band, l, nullptr, nullptr);
  p.res = describe_layer(P, l).res;   // (a residual from the chain's input has no address here)
  return lop::mbconv_describe(describe_layer(P, l - 1), p, name, size);
}

// Algorithmic work of that launch. A fused group: the three layers' operations on the rows
// it computes (the expand layer on the input rows the depthwise windows touch), and the
// bytes of the group's input rows, output rows, residual and weights only.
void launch_work(const lop_plan_t* P, int band, int l, double* flop, double* bytes) {
  const lop::Tables& t = P->t;
  const Fusion& F = band_fusion(P);
  const lop_rows_t r = launch_rows(P, F, band, l);
  *flop = 0.0;
  *bytes = 0.0;
  if (r.hi <= r.lo) return;
  if (F.head[l] < 0) {
    *flop = t.layer_flop(l, r.hi - r.lo);
    *bytes = t.layer_bytes(band, l);
    return;
  }
  if (ends_convpool(F, l)) {
    // the conv's operations on the rows under the windows plus the comparisons; bytes of the conv's
    // input rows and weights and of the pooled rows only
    const int h = F.head[l];
    const lop::LayerInfo &C = t.layers[h], &Q = t.layers[l];
    const lop_rows_t rd = t.bands[band].reads[h];
    const lop_rows_t cr = t.bands[band].compute[h];
    *flop = t.layer_flop(h, cr.hi - cr.lo) + t.layer_flop(l, r.hi - r.lo);
    const double e = (double)t.esz();
    *bytes = e * Q.n * ((double)(rd.hi - rd.lo) * C.w_in * C.d.c_in + (double)(r.hi - r.lo) * Q.w_out * Q.d.c_out) +
             e * (double)C.d.c_out * C.d.c_in * C.d.kh * C.d.kw;
    return;
  }
  const int h = F.head[l], m = h + 1;
  const lop::LayerInfo &E = t.layers[h], &D = t.layers[m], &Q = t.layers[l];
  const int in_lo = std::max(r.lo * D.d.sh - D.d.ph, 0);
  const int in_hi = std::min((r.hi - 1) * D.d.sh - D.d.ph + D.d.kh, D.h_in);
  const int rows_e = std::max(in_hi - in_lo, 0);
  *flop = t.layer_flop(l, r.hi - r.lo) + t.layer_flop(m, r.hi - r.lo) + t.layer_flop(h, rows_e);
  const double e = (double)t.esz();
  double b = e * Q.n * ((double)rows_e * E.w_in * E.d.c_in + (double)(r.hi - r.lo) * Q.w_out * Q.d.c_out);
  if (Q.d.residual_from != LOP_NO_RESIDUAL) b += e * Q.n * (double)(r.hi - r.lo) * Q.w_out * Q.d.c_out;
  b += e * ((double)E.d.c_out * E.d.c_in + 9.0 * D.d.c_out + (double)Q.d.c_out * Q.d.c_in);
  *bytes = b;
}

void* device_view_of_host(lop_plan_t* P, void* h_out);

// Small outputs (of a band, or of a chain whose bands run as merged launches) leave through the
// last layer's own stores: its kernel writes every element to the device tensor and to the mapped
// host buffer, so there is no copy launch to wait for on the lane. Larger outputs keep the paced copy kernel (stores over PCIe from a
// whole grid hold up the HBM writes of the kernels beside them: the 720p chain in reuse mode, 1.8 MB
// out, 90 us with the last layer's own stores, 72 with the copy kernel behind it, 60 without a copy).
constexpr size_t kDirectHostStoreMax = 256 * 1024;
// Workgroups of a band copy that shares the chip with kernels: its stores are paced by the link, and
// many of them in flight hold up the kernels beside the copy, first of all those on the compute units
// that the copy's workgroups share. Two workgroups of 512 move as much as four of 256 (about 30 GB/s),
// from half the compute units: 13 MB results of the inverted-residual chain 631 -> 591 us a chain,
// in reuse mode 505 -> 470; 1.8 MB ones the same. Eight and sixteen of 256 cost 698 and 785 us, one
// of 512 684 (the copies themselves then take longest), the copy engines 676.
constexpr int kCopyWorkgroups = 2;
constexpr size_t kCopyLaneMaxBytes = (size_t)64 << 20;

// Device view of h_out if the launches of one band (merged false), or those of the whole chain,
// can deliver their rows that way, else nullptr.
void* direct_host_target(lop_plan_t* P, int band, void* h_out, bool merged) {
  if (!h_out || (P->flags & (LOP_FLAG_NO_D2H | LOP_FLAG_DMA_COPY))) return nullptr;
  const lop::Tables& t = P->t;
  const int last = t.n_layers() - 1;
  const Fusion& F = merged ? P->fuse_chain : P->fuse_band;
  if (F.head[last] >= 0 && !ends_convpool(F, last)) return nullptr;
  const lop_rows_t r = t.bands[merged ? t.whole() : band].need[t.n_layers()];
  const size_t bytes = (size_t)t.in.n * (r.hi - r.lo) * t.row_elems(last) * t.esz();
  if (bytes == 0 || bytes > kDirectHostStoreMax) return nullptr;
  if (!ends_convpool(F, last) &&   // (the pooled launch stores to both destinations)
      !lop::stores_second_output(make_launch(P, band, last, nullptr, nullptr)))
    return nullptr;
  return device_view_of_host(P, h_out);
}

bool band_empty(const lop_plan_t* P, int band) {
  const lop_rows_t r = P->t.bands[band].need[P->t.n_layers()];
  return r.hi <= r.lo;
}

int enqueue_band_kernels(lop_plan_t* P, int band, const void* d_in, void* d_out, hipStream_t cs,
                         void* y2 = nullptr) {
  const int nl = P->t.n_layers();
  if (P->flags & LOP_FLAG_POISON_SCRATCH) {
    // Debug aid: every scratch byte the band could read is NaN (all bits set, in both storage
    // types) unless this band's own launches write it first, so a kernel that reads a row outside
    // the intervals the plan gave it shows up in the output. In reuse mode earlier bands' rows
    // are read on purpose: the slabs are poisoned once, before the chain's first band.
    bool first = true;
    for (int b = 0; b < band; ++b) first = first && band_empty(P, b);
    if (!P->t.reuse || first)
      LOP_HIP(lop::launch_fill_words(P->arena_of(band), align_up(P->arena_bytes, 256), 0xFFFFFFFFu, cs));
    LOP_HIP(lop::launch_fill_words(P->ws_of(band), P->conv_ws_bytes / 16 * 16, 0xFFFFFFFFu, cs));
  }
  for (int l = 0; l < nl; ++l)
    LOP_HIP(launch_layer(P, P->fuse_band, band, l, d_in, d_out, cs, nullptr, l == nl - 1 ? y2 : nullptr));
  return LOP_OK;
}

// Device-side address of a pinned, mapped host buffer, or nullptr if the buffer is not
// such memory. Looked up once per pointer.
void* device_view_of_host(lop_plan_t* P, void* h_out) {
  for (const auto& e : P->host_views)
    if (e.first == h_out) return e.second;
  void* dev = nullptr;
  hipPointerAttribute_t attr;
  if (hipPointerGetAttributes(&attr, h_out) == hipSuccess) {
    if (attr.type == hipMemoryTypeHost && attr.devicePointer) dev = attr.devicePointer;
  } else {
    (void)hipGetLastError();  // pageable memory: clear the sticky error, use the DMA path
  }
  if (P->host_views.size() >= 16) P->host_views.erase(P->host_views.begin());
  P->host_views.emplace_back(h_out, dev);
  return dev;
}

// Copy the final rows of a band (t.whole(): all rows) of every image to the host buffer (same
// NHWC layout).
int enqueue_band_copy(lop_plan_t* P, int band, const void* d_out, void* h_out, hipStream_t s) {
  const lop::Tables& t = P->t;
  const lop_rows_t r = t.bands[band].need[t.n_layers()];
  if (r.hi <= r.lo) return LOP_OK;
  const lop::LayerInfo& L = t.layers.back();
  const size_t row_b = (size_t)t.row_elems(t.n_layers() - 1) * t.esz();
  const size_t img_b = row_b * L.h_out;
  const bool all = r.hi - r.lo == L.h_out;   // (the images' rows are then one contiguous run)
  const int n = all ? 1 : t.in.n;
  const size_t off = row_b * r.lo, len = row_b * (r.hi - r.lo) * (all ? t.in.n : 1);
  // Mapped pinned host memory is written by a small kernel on the copy stream (no DMA
  // set-up cost per band, and it can be captured like any kernel); a plan made with
  // LOP_FLAG_DMA_COPY goes through the runtime's copy engines instead. Host memory that is
  // not pinned is refused (the boundary asks for pinned memory: an asynchronous copy into
  // pageable memory is staged by the runtime and is neither asynchronous nor cheap).
  void* mapped = device_view_of_host(P, h_out);
  if (!mapped) return LOP_ERR_INVALID_ARG;
  if (P->flags & LOP_FLAG_DMA_COPY) mapped = nullptr;
  if (mapped) {
    LOP_HIP(lop::launch_copy_rows((char*)mapped + off, (const char*)d_out + off, img_b, len, n, s, kCopyWorkgroups));
    return LOP_OK;
  }
  if (n == 1) {
    LOP_HIP(hipMemcpyAsync((char*)h_out + off, (const char*)d_out + off, len,
                           hipMemcpyDeviceToHost, s));
  } else {
    LOP_HIP(hipMemcpy2DAsync((char*)h_out + off, img_b, (const char*)d_out + off, img_b, len, n,
                             hipMemcpyDeviceToHost, s));
  }
  return LOP_OK;
}

int ensure_timing_events(lop_plan_t* P) {
  if (!P->ev_c0.empty()) return LOP_OK;
  const int nb = P->t.n_bands;
  for (auto* v : {&P->ev_c0, &P->ev_c1, &P->ev_d0, &P->ev_d1}) {
    v->assign(nb, nullptr);
    for (int b = 0; b < nb; ++b) LOP_HIP(hipEventCreate(&(*v)[b]));
  }
  LOP_HIP(hipEventCreate(&P->ev_t0));
  LOP_HIP(hipEventCreate(&P->ev_t1));
  return LOP_OK;
}

int setup_device(lop_plan_t* P) {
  LOP_HIP(hipGetDevice(&P->device));
  LOP_HIP(resolve_static_scratch(P->device));
  int rc = upload_weights(P);
  if (rc != LOP_OK) return rc;
  const int nb = P->t.n_bands;
  int live = 0;
  for (int b = 0; b < nb; ++b) live += band_empty(P, b) ? 0 : 1;
  int want = (int)((P->flags >> 8) & 0xff);
  if (want == 0) {
    want = LOP_DEFAULT_LANES;
    // Slabs that fill most of the 256 MB Infinity Cache by themselves: two lanes, not four, whose launches would only
    // push each other's rows out of it. Where a lane is needed for copies, four are better all the same. (Inverted-residual
    // chain layer by layer, us a call with four lanes and with two: 156 MiB a lane 1 308 and 1 384, 170 MiB 1 432 and 1 498, 188 MiB 1 588
    // and 1 618 or 1 609 and 1 606, 208 MiB 1 777 and 1 756, 219 MiB 1 865 and 1 832, 228 MiB 1 948 and 1 916, 250 MiB 2 152 and 2 050.)
    if (P->sched == ChainSched::kPerBand && !P->t.reuse && P->arena_bytes > kLaneSlabsMax && (P->flags & LOP_FLAG_NO_D2H)) want = 2;
  }
  // (chains that run on one lane each rotate over all of them, however few bands they have)
  const bool by_chain = P->t.reuse || P->sched != ChainSched::kPerBand;
  const int n_lanes = by_chain ? std::max(1, want) : std::max(1, std::min(want, live));
  P->lanes.assign(n_lanes, Lane{});
  // Long band copies (stores into host memory, paced by the link) get a lane of their own.
  // On a compute lane a copy holds up that lane's next band, and because the bands are equal
  // the lanes reach their copies together: all of them copy at once, at the link's rate, with
  // nothing computing beside them, and then all compute at once with the link idle.
  size_t longest_copy = 0, all_copies = 0;
  for (int b = 0; b < nb; ++b) {
    const lop_rows_t r = P->t.bands[b].need[P->t.n_layers()];
    if (r.hi <= r.lo) continue;
    const size_t bytes = (size_t)P->t.in.n * (r.hi - r.lo) * P->t.row_elems(P->t.n_layers() - 1) * P->t.esz();
    longest_copy = std::max(longest_copy, bytes);
    all_copies += bytes;
  }
  // Independent bands only: in reuse mode a lane holds a whole chain, and three chains in
  // flight plus a copy lane measured slower than four chains that copy on their own lanes.
  // Not for chains whose result is so large that the copies, one after another at the copy
  // kernel's 30 GB/s, would take longer than the kernels (a matrix product chain with 134 MB of
  // output per call: 215 calls/s with the copy lane, 350 with copies on every lane, which
  // together reach the link's rate). The plan does not know the kernels' time; the bound on the
  // bytes stands for it.
  P->copy_lane = !by_chain && n_lanes >= 3 && longest_copy > kDirectHostStoreMax &&
                 all_copies <= kCopyLaneMaxBytes &&
                 !(P->flags & (LOP_FLAG_NO_D2H | LOP_FLAG_DMA_COPY));
  for (Lane& L : P->lanes) {
    const bool computes = !P->copy_lane || &L != &P->lanes.back();
    if (P->arena_bytes && computes) LOP_HIP(lop::dev_alloc(&L.arena, align_up(P->arena_bytes, 256)));
    if (P->conv_ws_bytes && computes) {
      LOP_HIP(lop::dev_alloc(&L.conv_ws, P->conv_ws_bytes));
    }
    LOP_HIP(hipStreamCreateWithFlags(&L.stream, hipStreamNonBlocking));
    LOP_HIP(hipStreamCreateWithFlags(&L.copy, hipStreamNonBlocking));
    LOP_HIP(hipEventCreateWithFlags(&L.ev_join, hipEventDisableTiming));
  }
  LOP_HIP(hipStreamCreateWithFlags(&P->s_main, hipStreamNonBlocking));
  LOP_HIP(hipStreamCreateWithFlags(&P->s_copy, hipStreamNonBlocking));
  LOP_HIP(hipEventCreateWithFlags(&P->ev_fork, hipEventDisableTiming));
  LOP_HIP(hipEventCreateWithFlags(&P->ev_copy_tail, hipEventDisableTiming));
  P->ev_done.assign(nb, nullptr);
  P->ev_copied.assign(nb, nullptr);
  P->copied_valid.assign(nb, 0);
  for (auto& e : P->ev_done) LOP_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  for (auto& e : P->ev_copied) LOP_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  LOP_HIP(hipDeviceSynchronize());
  return LOP_OK;
}

// Kernels of one band on stream `cs`, then (optionally) its device-to-host copy on the
// copy stream, gated by the band's "kernels finished" event.
int enqueue_band(lop_plan_t* P, int band, const void* d_in, void* d_out, void* h_out,
                 hipStream_t cs, hipStream_t ds, bool timing, bool capturing = false) {
  // the band's rows of d_out may still be in flight to the host from an earlier call
  if (P->copied_valid[band] && !capturing)
    LOP_HIP(hipStreamWaitEvent(cs, P->ev_copied[band], 0));
  if (timing) LOP_HIP(hipEventRecord(P->ev_c0[band], cs));
  void* const direct = direct_host_target(P, band, h_out, false);
  int rc = enqueue_band_kernels(P, band, d_in, d_out, cs, direct);
  if (rc != LOP_OK) return rc;
  if (timing) LOP_HIP(hipEventRecord(P->ev_c1[band], cs));
  if (direct) {  // the rows are on their way already: nothing to copy, nothing to wait for
    if (timing) {
      LOP_HIP(hipEventRecord(P->ev_d0[band], cs));
      LOP_HIP(hipEventRecord(P->ev_d1[band], cs));
    }
    if (!capturing) {
      LOP_HIP(hipEventRecord(P->ev_copied[band], cs));
      P->copied_valid[band] = 1;
    }
  } else if (h_out && !(P->flags & LOP_FLAG_NO_D2H)) {
    if (ds != cs) {  // stream order already gates a copy on the kernels' own stream
      LOP_HIP(hipEventRecord(P->ev_done[band], cs));
      LOP_HIP(hipStreamWaitEvent(ds, P->ev_done[band], 0));
    }
    if (timing) LOP_HIP(hipEventRecord(P->ev_d0[band], ds));
    rc = enqueue_band_copy(P, band, d_out, h_out, ds);
    if (rc != LOP_OK) return rc;
    if (timing) LOP_HIP(hipEventRecord(P->ev_d1[band], ds));
    if (!capturing) {
      LOP_HIP(hipEventRecord(P->ev_copied[band], ds));
      P->copied_valid[band] = 1;
    }
  }
  return LOP_OK;
}

// Fork the lanes from `ms`, enqueue every band, join the lanes back into `ms`.
int enqueue_chain(lop_plan_t* P, const void* d_in, void* d_out, void* h_out, hipStream_t ms,
                  bool timing, bool capturing) {
  hipStream_t ds = P->s_copy;
  LOP_HIP(hipEventRecord(P->ev_fork, ms));
  for (Lane& L : P->lanes) LOP_HIP(hipStreamWaitEvent(L.stream, P->ev_fork, 0));
  bool copied = false;
  for (int b = 0; b < P->t.n_bands; ++b) {
    if (band_empty(P, b)) continue;
    // With several lanes a band's copy follows its kernels on the lane's own stream and
    // overlaps the other lanes' kernels; a single lane needs the separate copy stream to
    // overlap band b's copy with band b+1's kernels.
    hipStream_t cs = P->lane_of(b).stream;
    int rc = enqueue_band(P, b, d_in, d_out, h_out, cs, P->n_lanes() > 1 ? cs : ds, timing,
                          capturing);
    if (rc != LOP_OK) return rc;
    copied = copied || (h_out && !(P->flags & LOP_FLAG_NO_D2H));
  }
  // join: the main stream continues once every lane's kernels are done. Eagerly the
  // copies are not joined, so the last copy can run under whatever is enqueued next; a
  // captured graph has to join every stream it forked.
  for (Lane& L : P->lanes) {
    LOP_HIP(hipEventRecord(L.ev_join, L.stream));
    LOP_HIP(hipStreamWaitEvent(ms, L.ev_join, 0));
  }
  if (capturing && copied && P->n_lanes() == 1) {
    LOP_HIP(hipEventRecord(P->ev_copy_tail, ds));
    LOP_HIP(hipStreamWaitEvent(ms, P->ev_copy_tail, 0));
  }
  return LOP_OK;
}

// Bands of a reuse-mode chain, in order, on one lane.
int enqueue_chain_reuse(lop_plan_t* P, const void* d_in, void* d_out, void* h_out, bool timing,
                        bool capturing) {
  Lane& L = P->lanes[P->cur_lane];
  // With several lanes a band's copy follows its kernels on the lane and overlaps the
  // other lanes' chains (cross-stream edges inside a captured graph were measured to
  // serialise the lanes); a single lane uses its copy stream so that band b's copy
  // overlaps band b+1's kernels.
  hipStream_t ds = P->n_lanes() > 1 ? L.stream : L.copy;
  bool copied = false;
  for (int b = 0; b < P->t.n_bands; ++b) {
    if (band_empty(P, b)) continue;
    int rc = enqueue_band(P, b, d_in, d_out, h_out, L.stream, ds, timing, capturing);
    if (rc != LOP_OK) return rc;
    copied = copied || (h_out && !(P->flags & LOP_FLAG_NO_D2H));
  }
  if (capturing && copied && ds != L.stream) {  // a captured graph joins the stream it forked
    LOP_HIP(hipEventRecord(P->ev_copy_tail, ds));
    LOP_HIP(hipStreamWaitEvent(L.stream, P->ev_copy_tail, 0));
  }
  return LOP_OK;
}

// The descriptors of layer l's launch for bands [first, last) (heads: the conv of a conv + pooling
// group or the expand operator of an inverted-residual block, else empty).
void batched_group(const lop_plan_t* P, int l, int first, int last, const void* d_in, void* d_out, void* y2,
                   std::vector<lop::OpLaunch>* group, std::vector<lop::OpLaunch>* heads) {
  group->clear();
  heads->clear();
  const Fusion& F = P->fuse_chain;
  for (int b = first; b < last; ++b) {
    const lop_rows_t r = launch_rows(P, F, b, l);
    if (r.hi <= r.lo) continue;
    lop::OpLaunch head, o;
    if (F.head[l] < 0) {
      o = make_launch(P, b, l, d_in, d_out);
    } else {
      if (ends_convpool(F, l)) convpool_launches(P, b, l, d_in, d_out, &head, &o);
      else mbconv_launches(P, F.head[l], b, l, d_in, d_out, &head, &o);
      heads->push_back(head);
    }
    o.y2 = y2;
    group->push_back(o);
  }
}

// Layer l of bands [first, last): one launch (plus its finish kernel, if the reduction is cut) per
// kMaxBandsPerLaunch bands.
hipError_t launch_layer_batched(const lop_plan_t* P, int l, int first, int last, const void* d_in, void* d_out, hipStream_t cs,
                                lop::KernelEvents* ev, void* y2) {
  const Fusion& F = P->fuse_chain;
  if (F.away[l]) return hipSuccess;
  std::vector<lop::OpLaunch> group, heads;
  for (; first < last; first += lop::kMaxBandsPerLaunch) {
    batched_group(P, l, first, std::min(last, first + lop::kMaxBandsPerLaunch), d_in, d_out, y2, &group, &heads);
    const int n = (int)group.size();
    if (n == 0) continue;
    const hipError_t e = F.head[l] < 0 ? lop::launch_op_bands(group.data(), n, cs, ev)
                         : ends_convpool(F, l)
                             ? lop::launch_convpool_bands(heads.data(), group.data(), n, cs, ev)
                             : lop::launch_mbconv_bands(heads.data(), describe_layer(P, F.head[l] + 1), group.data(), n, cs, ev);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Kernel name and reduction slices of that launch (of a plan made with LOP_FLAG_BATCH_BANDS).
int describe_layer_batched(const lop_plan_t* P, int l, char* name, size_t size) {
  if (P->fuse_chain.away[l]) return 0;
  std::vector<lop::OpLaunch> group, convs;
  batched_group(P, l, 0, P->t.n_bands, nullptr, nullptr, nullptr, &group, &convs);
  if (group.empty()) return 0;
  if (ends_convpool(P->fuse_chain, l))
    return lop::convpool_describe_bands(convs.data(), group.data(), (int)group.size(), name, size);
  return lop::describe_op_bands(group.data(), (int)group.size(), name, size);
}

// The band a batched plan's launch of layer l is attributed to in per-band queries: the first
// band that computes rows of it (-1: nobody does).
int batched_owner(const lop_plan_t* P, int l) {
  for (int b = 0; b < P->t.n_bands; ++b) {
    const lop_rows_t r = launch_rows(P, P->fuse_chain, b, l);
    if (r.hi > r.lo) return b;
  }
  return -1;
}

// Scratch of a chain while it is enqueued: a lane's, or the static array's.
struct ChainScratch {
  lop_plan_t* P;
  ChainScratch(lop_plan_t* plan, void* arena, void* ws, bool alone) : P(plan) {
    P->arena_override = arena; P->ws_override = ws; P->alone = alone;
  }
  ~ChainScratch() { P->arena_override = nullptr; P->ws_override = nullptr; P->alone = false; }
};

// The same of a chain that runs on a lane's own scratch.
struct ChainAlone {
  lop_plan_t* P;
  ChainAlone(lop_plan_t* plan, bool alone) : P(plan) { P->alone = alone; }
  ~ChainAlone() { P->alone = false; }
};

// Whether layers l and l + 1 are a convolution and the 1 x 1 shortcut beside it, which a merged chain computes
// in one launch where a kernel takes both (a launch more costs a chain 4 us, and the small
// shortcut leaves most of the chip idle). The second one's output is then written while the first is computed, so
// neither may read anything else: every buffer still needed then keeps its memory.
bool siblings(const lop_plan_t* P, int l) {
  const lop::Tables& t = P->t;
  if (l + 2 >= t.n_layers()) return false;
  const lop_layer_t &a = t.layers[l].d, &b = t.layers[l + 1].d;
  if (a.op != LOP_CONV2D || b.op != LOP_CONV2D || a.input_from != b.input_from || a.kh != 3 || b.kh != 1) return false;
  if (a.residual_from != LOP_NO_RESIDUAL || b.residual_from != LOP_NO_RESIDUAL || last_reader(P, l) <= l + 1) return false;
  const Fusion& F = P->fuse_chain;
  return !F.away[l] && !F.away[l + 1] && F.head[l] < 0 && F.head[l + 1] < 0 && !(P->flags & LOP_FLAG_NO_FUSE);
}

// Whether layers l and l + 1 are two convolutions of which the second is the only reader of the first, which a merged
// chain computes in one launch for bands [first, last) where a kernel takes both. The rows between them are then in no buffer.
// (What the launch would be refused for is looked at here as far as it is cheap: a refused one's descriptors are made for nothing. Between
// two buffers of the chain the second layer's output lies, as a rule, where the first one's input does.)
bool pair(const lop_plan_t* P, int l, int first, int last) {
  const lop::Tables& t = P->t;
  if (l + 1 >= t.n_layers() || (P->flags & LOP_FLAG_NO_FUSE)) return false;
  const lop_layer_t &a = t.layers[l].d, &b = t.layers[l + 1].d;
  if (a.op != LOP_CONV2D || b.op != LOP_CONV2D || b.input_from != l) return false;
  for (const lop_layer_t* d : {&a, &b})
    if (d->c_in != lop::kPairChannels || d->c_out != lop::kPairChannels || d->kh != 3 || d->kw != 3 || d->residual_from != LOP_NO_RESIDUAL) return false;
  const Fusion& F = P->fuse_chain;
  if (F.away[l] || F.away[l + 1] || F.head[l] >= 0 || F.head[l + 1] >= 0) return false;
  if (const int x = a.input_from; x >= 0 && l + 1 < t.n_layers() - 1) {   // (the bands' slabs of a layer lie one behind the other)
    auto end = [&](const lop::Slab& s) { return (const char*)s.ptr + (size_t)s.n * s.rows * s.w * s.c * t.esz(); };
    const lop::Slab from = slab_of(P, first, x, nullptr, nullptr), to = slab_of(P, first, l + 1, nullptr, nullptr);
    if ((const char*)from.ptr < end(slab_of(P, last - 1, l + 1, nullptr, nullptr)) && (const char*)to.ptr < end(slab_of(P, last - 1, x, nullptr, nullptr)))
      return false;
  }
  return last_reader(P, l) == l + 1;
}

// The last layer of the launch that a first layer l and the convolution behind it, its only reader, share where a kernel
// takes both (l + 1, or l + 2 if that convolution's pooling is part of its launch), or -1.
int front_end(const lop_plan_t* P, int l) {
  const lop::Tables& t = P->t;
  const int nl = t.n_layers();
  if (t.layers[l].d.c_in != 3 || l + 1 >= nl || (P->flags & LOP_FLAG_NO_FUSE)) return -1;
  for (int j = 0; j < nl; ++j)
    if ((j != l + 1 && t.layers[j].d.input_from == l) || t.layers[j].d.residual_from == l) return -1;
  const lop_layer_t &a = t.layers[l].d, &b = t.layers[l + 1].d;
  const Fusion& F = P->fuse_chain;
  if (a.op != LOP_CONV2D || b.op != LOP_CONV2D || b.input_from != l || F.away[l] || F.head[l] >= 0 || F.head[l + 1] >= 0) return -1;
  if (!F.away[l + 1]) return l + 1;
  return l + 2 < nl && F.head[l + 2] == l + 1 ? l + 2 : -1;
}

// The kernels of a chain whose launches are merged over the bands (kGrouped, kWhole), on one
// stream, with the scratch set by the caller. y2: where the last launch also stores its rows.
int enqueue_merged_kernels(lop_plan_t* P, const void* d_in, void* d_out, hipStream_t cs, void* y2) {
  const int nl = P->t.n_layers(), whole = P->t.whole();
  // (kept: bytes at the arena's beginning that earlier passes have written)
  auto begin_pass = [&](size_t kept) -> int {
    if (!(P->flags & LOP_FLAG_POISON_SCRATCH)) return LOP_OK;
    LOP_HIP(lop::launch_fill_words((char*)P->arena_of(0) + kept, align_up(P->arena_bytes, 256) - kept, 0xFFFFFFFFu, cs));
    LOP_HIP(lop::launch_fill_words(P->ws_of(0), P->conv_ws_bytes / 16 * 16, 0xFFFFFFFFu, cs));
    return LOP_OK;
  };
  const int nb = P->t.n_bands, n = P->t.in.n;
  const size_t out_bytes = (size_t)P->t.layers.back().h_out * P->t.row_elems(nl - 1) * P->t.esz();   // of one image
  // layers [first, last) of all rows ...
  auto whole_layers = [&](int first, int last, void* second) -> int {
    for (int l = first; l < last; ++l) {
      if (const int e = front_end(P, l); e > 0 && e < last) {
        const lop::OpLaunch a = make_launch(P, whole, l, d_in, d_out);
        lop::OpLaunch c = make_launch(P, whole, l + 1, d_in, d_out), q = make_launch(P, whole, e, d_in, d_out);
        c.y2 = q.y2 = e == nl - 1 ? second : nullptr;
        bool taken;
        LOP_HIP(lop::launch_front(&a, &c, e > l + 1 ? &q : nullptr, 1, cs, &taken));
        if (taken) {
          l = e;
          continue;
        }
      }
      if (l + 1 < last && pair(P, l, whole, whole + 1)) {
        const lop::OpLaunch a = make_launch(P, whole, l, d_in, d_out);
        lop::OpLaunch q = make_launch(P, whole, l + 1, d_in, d_out);
        q.y2 = l + 1 == nl - 1 ? second : nullptr;
        if (lop::pair_applies(&a, &q, 1)) {
          LOP_HIP(lop::launch_pair(&a, &q, 1, cs));
          ++l;
          continue;
        }
      }
      if (l + 1 < last && siblings(P, l)) {
        const lop::OpLaunch a = make_launch(P, whole, l, d_in, d_out), q = make_launch(P, whole, l + 1, d_in, d_out);
        if (a.out_hi > a.out_lo && lop::siblings_apply(&a, &q, 1)) {
          LOP_HIP(lop::launch_siblings(&a, &q, 1, cs));
          ++l;
          continue;
        }
      }
      LOP_HIP(launch_layer(P, P->fuse_chain, whole, l, d_in, d_out, cs, nullptr, l == nl - 1 ? second : nullptr));
    }
    return LOP_OK;
  };
  // ... and of bands [b, end)
  auto grouped_layers = [&](int first, int last, int b, int end, void* second) -> int {
    const bool together = end - b <= lop::kMaxBandsPerLaunch;
    for (int l = first; l < last; ++l) {
      if (const int e = front_end(P, l); e > 0 && e < last && together) {
        std::vector<lop::OpLaunch> as, convs, qs, none;
        batched_group(P, l, b, end, d_in, d_out, nullptr, &as, &none);
        batched_group(P, e, b, end, d_in, d_out, e == nl - 1 ? second : nullptr, &qs, &convs);
        const bool pooled = e > l + 1;
        bool taken = false;
        if (as.size() == qs.size())
          LOP_HIP(lop::launch_front(as.data(), pooled ? convs.data() : qs.data(), pooled ? qs.data() : nullptr, (int)as.size(), cs, &taken));
        if (taken) {
          l = e;
          continue;
        }
      }
      if (l + 1 < last && together && pair(P, l, b, end)) {
        std::vector<lop::OpLaunch> as, qs, none;
        batched_group(P, l, b, end, d_in, d_out, nullptr, &as, &none);
        batched_group(P, l + 1, b, end, d_in, d_out, l + 1 == nl - 1 ? second : nullptr, &qs, &none);
        if (as.size() == qs.size() && lop::pair_applies(as.data(), qs.data(), (int)as.size())) {
          LOP_HIP(lop::launch_pair(as.data(), qs.data(), (int)as.size(), cs));
          ++l;
          continue;
        }
      }
      if (l + 1 < last && together && siblings(P, l)) {
        std::vector<lop::OpLaunch> as, qs, none;
        batched_group(P, l, b, end, d_in, d_out, nullptr, &as, &none);
        batched_group(P, l + 1, b, end, d_in, d_out, nullptr, &qs, &none);
        if ((int)as.size() == end - b && qs.size() == as.size() && lop::siblings_apply(as.data(), qs.data(), end - b)) {
          LOP_HIP(lop::launch_siblings(as.data(), qs.data(), end - b, cs));
          ++l;
          continue;
        }
      }
      LOP_HIP(launch_layer_batched(P, l, b, end, d_in, d_out, cs, nullptr, l == nl - 1 ? second : nullptr));
    }
    return LOP_OK;
  };
  const int in_passes = P->cut < 0 ? nl : P->cut + 1;
  for (int i = 0; i < n; i += P->images) {
    void* const second = y2 ? (char*)y2 + i * out_bytes : nullptr;
    const int images = std::min(P->images, n - i);
    for (int b = 0; b < nb; b += P->group) {
      const int end = std::min(nb, b + P->group);
      const bool part = P->sched == ChainSched::kWhole && P->group < nb;   // (of a chain whose layers keep to their rows)
      const lop_rows_t rows = part ? pass_rows(P, b, end) : lop_rows_t{0, 0};
      if (part && rows.hi <= rows.lo) continue;
      if (const int rc = begin_pass(i + b > 0 ? P->cut_bytes : 0); rc != LOP_OK) return rc;
      const ChainPass pass(P, i, images, rows);
      const int rc = P->sched == ChainSched::kWhole ? whole_layers(0, in_passes, second) : grouped_layers(0, in_passes, b, end, second);
      if (rc != LOP_OK) return rc;
    }
  }
  if (in_passes == nl) return LOP_OK;
  if (const int rc = begin_pass(P->cut_bytes); rc != LOP_OK) return rc;
  const ChainPass pass(P, 0, n);
  return P->sched == ChainSched::kWhole ? whole_layers(in_passes, nl, y2) : grouped_layers(in_passes, nl, 0, nb, y2);
}

// The kernels of a chain whose launches are merged over the bands (Sec. IV-D operation batching), on
// one lane's scratch and on stream `cs`: per layer one launch for the rows of all bands. direct:
// where the last one also stores its rows (device view of the host buffer), or nullptr. alone: the chain is for a caller's
// stream (a graph is captured as its first caller wants it; what that changes is no bit of the result).
int enqueue_chain_merged(lop_plan_t* P, Lane& L, const void* d_in, void* d_out, void* direct, hipStream_t cs, bool alone) {
  ChainScratch scratch(P, L.arena, L.conv_ws, alone);
  return enqueue_merged_kernels(P, d_in, d_out, cs, direct);
}

// Orders stream `s` behind everything that may still use the lane's scratch and notes that `s` uses it
// next. waited (optional): the event that `s` waited for last, so that lanes sharing one cost one wait.
int take_lane(Lane& L, hipStream_t s, hipEvent_t* waited = nullptr) {
  if (L.user || s != L.stream) {   // (else stream order does it)
    if (!L.user) {
      LOP_HIP(hipEventRecord(L.ev_join, L.stream));
      L.left = L.ev_join;
    }
    if (!waited || *waited != L.left) LOP_HIP(hipStreamWaitEvent(s, L.left, 0));
    if (waited) *waited = L.left;
  }
  L.user = s == L.stream ? nullptr : s;
  return LOP_OK;
}

// Marks the end of a use of the lane's scratch on a stream that is not the lane's own.
int leave_lane(Lane& L) {
  if (!L.user) return LOP_OK;
  LOP_HIP(hipEventRecord(L.ev_join, L.user));
  L.left = L.ev_join;
  return LOP_OK;
}

// ... and of a use of all lanes by one stream.
int leave_lanes(lop_plan_t* P) {
  const int rc = leave_lane(P->lanes[0]);
  for (Lane& L : P->lanes) L.left = P->lanes[0].left;
  return rc;
}

// The bands of lane `lane` of an independent-mode chain, in order, on that lane's stream.
int enqueue_lane(lop_plan_t* P, int lane, const void* d_in, void* d_out, void* h_out, bool capturing) {
  hipStream_t cs = P->lanes[lane].stream;
  for (int b = lane; b < P->t.n_bands; b += P->n_lanes()) {
    if (band_empty(P, b)) continue;
    int rc = enqueue_band(P, b, d_in, d_out, h_out, cs, cs, false, capturing);
    if (rc != LOP_OK) return rc;
  }
  return LOP_OK;
}

hipGraphExec_t find_graph(const lop_plan_t* P, const void* d_in, const void* d_out, const void* h_out, int lane,
                          int band) {
  for (const auto& g : P->graphs)
    if (g.d_in == d_in && g.d_out == d_out && g.h_out == h_out && g.lane == lane && g.band == band) return g.exec;
  return nullptr;
}

// Instantiates what was captured (rc, e: how enqueueing and ending the capture went) and keeps it.
int keep_graph(lop_plan_t* P, int rc, hipError_t e, hipGraph_t graph, const void* d_in, void* d_out, void* h_out,
               int lane, int band, hipGraphExec_t* exec) {
  if (rc != LOP_OK) {
    if (graph) (void)hipGraphDestroy(graph);
    return rc;
  }
  if (e != hipSuccess) return hip_fail(e);
  e = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) return hip_fail(e);
  if (P->graphs.size() >= 128) {  // bounded cache: drop the oldest
    (void)hipGraphExecDestroy(P->graphs.front().exec);
    P->graphs.erase(P->graphs.begin());
  }
  P->graphs.push_back({d_in, d_out, h_out, lane, band, *exec});
  return LOP_OK;
}

// lane_only >= 0 (independent mode): the graph holds that lane's bands only and runs on the
// lane's stream `ms`; -1: the whole chain forked from and joined into `ms`.
// band_only >= 0: the graph holds that band's kernels and nothing else (its copy is the
// caller's business).
int launch_graph(lop_plan_t* P, const void* d_in, void* d_out, void* h_out, hipStream_t ms,
                 int lane_only = -1, int band_only = -1) {
  const int lane = lane_only >= 0 ? lane_only : P->t.reuse ? P->cur_lane : -1;
  // an eager run may still have copies of the output rows in flight (on a copy stream that the
  // graph's stream is not ordered behind): a replay, and the first capture, wait for them
  for (int b = 0; b < P->t.n_bands; ++b)
    if (P->copied_valid[b] && (band_only < 0 || b == band_only)) {
      LOP_HIP(hipStreamWaitEvent(ms, P->ev_copied[b], 0));
      P->copied_valid[b] = 0;
    }
  if (hipGraphExec_t exec = find_graph(P, d_in, d_out, h_out, lane, band_only)) {
    LOP_HIP(hipGraphLaunch(exec, ms));
    return LOP_OK;
  }
  if (h_out) (void)device_view_of_host(P, h_out);  // query before capture starts
  hipGraph_t graph = nullptr;
  LOP_HIP(hipStreamBeginCapture(ms, hipStreamCaptureModeThreadLocal));
  int rc = band_only >= 0 ? enqueue_band_kernels(P, band_only, d_in, d_out, ms)
           : P->t.reuse  ? enqueue_chain_reuse(P, d_in, d_out, h_out, false, true)
           : lane_only >= 0 ? enqueue_lane(P, lane_only, d_in, d_out, h_out, true)
                            : enqueue_chain(P, d_in, d_out, h_out, ms, false, true);
  hipError_t e = hipStreamEndCapture(ms, &graph);
  hipGraphExec_t exec = nullptr;
  rc = keep_graph(P, rc, e, graph, d_in, d_out, h_out, lane, band_only, &exec);
  if (rc != LOP_OK) return rc;
  LOP_HIP(hipGraphLaunch(exec, ms));
  return LOP_OK;
}

// What a merged chain's launches (by layers: a pair counts as two; finish kernels aside) cost the host, in sixteenths of a launch of
// one band: each further band of a launch is one more, for the descriptor and the parameters it makes.
struct MergedCost { long launches = 0, host = 0; };
MergedCost merged_cost(const lop_plan_t* P) {
  const int nl = P->t.n_layers(), nb = P->t.n_bands, n = P->t.in.n, in_passes = P->cut < 0 ? nl : P->cut + 1;
  MergedCost c;
  auto add = [&](int bands, long times) {
    const bool grouped = P->sched == ChainSched::kGrouped;
    const long launches = grouped ? (bands + lop::kMaxBandsPerLaunch - 1) / lop::kMaxBandsPerLaunch : 1;
    c.launches += launches * times;
    c.host += (launches * 16 + (grouped ? bands : 0)) * times;
  };
  for (int l = 0; l < nl; ++l) {
    if (P->fuse_chain.away[l]) continue;
    if (l >= in_passes) { add(nb, 1); continue; }
    for (int b = 0; b < nb; b += P->group) add(std::min(P->group, nb - b), (n + P->images - 1) / P->images);
  }
  return c;
}
// Merged chains of few launches are enqueued by every call, also where the plan asks for graphs: a graph's launch costs 12 to 20 us of
// host time however few nodes it has, one of a kernel 3 to 7, and a stream gets through a graph's kernels 6 us later. us a call, graph ->
// kernels, with calls in flight, on one caller's stream, and alone: one launch (two layers of 16 channels) 14.0 -> 4.8, 15.8 -> 8.5, 33 -> 18;
// layers of 3000 x 512 x 512 (bf16, a launch for all rows): two 18.7 -> 10.4, 26.4 -> 19.4, 38 -> 28, four 23.3 -> 21.4, 42.3 -> 36.3, 50 -> 45, but
// five 22.2 -> 22.9, 52.7 -> 45.9, 61 -> 55. With bands in the launches (3 x 3, 32 channels, 64 x 64 or 160 x 160 pixels; fp32's parameters are the
// larger) the line for calls in flight lies earlier: eight bands, three launches 16.3 -> 15.7 to 25.4 -> 19.8, four 17.3 -> 19.5, 20.0 -> 21.9;
// sixteen, two 20.0 -> 11.8 to 23.0 -> 14.3, three 17.1 -> 20.9 to 25.3 -> 24.2, four 24.4 -> 26.4. On a caller's stream what a graph holds up
// counts for more: four of eight bands 34.0 -> 29.3 and 50.3 -> 44.3 (160 x 160), 28.2 -> 28.6 and 28.6 -> 31.6 (64 x 64, where the host is all there
// is), three of sixteen 30.3 -> 24.8, 44.1 -> 37.5, 25.7 -> 24.7 and 25.2 -> 30.1; four of sixteen 30.7 -> 33.4.
constexpr long kEagerLaunches = 4, kEagerHost = 80, kEagerHostAlone = 112;
bool enqueued_by_every_call(const lop_plan_t* P, bool alone) {
  const MergedCost c = merged_cost(P);
  return c.launches <= kEagerLaunches && c.host <= (alone ? kEagerHostAlone : kEagerHost);
}

// A merged chain's kernels as a graph: captured on lane `lane`'s own stream (with that lane's
// scratch), replayed on `s`.
int launch_graph_merged(lop_plan_t* P, int lane, const void* d_in, void* d_out, void* direct, hipStream_t s) {
  Lane& L = P->lanes[lane];
  hipGraphExec_t exec = find_graph(P, d_in, d_out, direct, lane, -1);
  if (!exec) {
    hipGraph_t graph = nullptr;
    LOP_HIP(hipStreamBeginCapture(L.stream, hipStreamCaptureModeThreadLocal));
    int rc = enqueue_chain_merged(P, L, d_in, d_out, direct, L.stream, s != L.stream);
    const hipError_t e = hipStreamEndCapture(L.stream, &graph);
    rc = keep_graph(P, rc, e, graph, d_in, d_out, direct, lane, -1, &exec);
    if (rc != LOP_OK) return rc;
  }
  LOP_HIP(hipGraphLaunch(exec, s));
  return LOP_OK;
}

// One merged chain: picks a lane, orders the chain behind what it must not overtake and enqueues
// it on the caller's stream, or on the lane's own where there is none to order against (chains
// of consecutive calls then overlap).
int run_merged(lop_plan_t* P, const void* d_in, void* d_out, void* h_out, hipStream_t user, bool timing) {
  int lane = P->next_lane;
  if (user)   // (a caller's stream runs its chains one after another: it stays on the lane it used last)
    for (int k = 0; k < (int)P->lanes.size(); ++k)
      if (P->lanes[k].user == user) lane = k;
  if (lane == P->next_lane) P->next_lane = (P->next_lane + 1) % (int)P->lanes.size();
  P->cur_lane = lane;
  Lane& L = P->lanes[lane];
  hipStream_t s = user ? user : L.stream;
  int rc = take_lane(L, s);
  if (rc != LOP_OK) return rc;
  const int nb = P->t.n_bands;
  for (int b = 0; b < nb; ++b)
    if (P->copied_valid[b]) {  // copies of single bands of an earlier call that may still read d_out
      LOP_HIP(hipStreamWaitEvent(s, P->ev_copied[b], 0));
      P->copied_valid[b] = 0;
    }
  auto stamp = [&](std::vector<hipEvent_t>& ev) -> int {   // (the bands of a merged chain start and end together)
    if (timing)
      for (int b = 0; b < nb; ++b)
        if (!band_empty(P, b)) LOP_HIP(hipEventRecord(ev[b], s));
    return LOP_OK;
  };
  if (timing) LOP_HIP(hipEventRecord(P->ev_t0, s));
  if ((rc = stamp(P->ev_c0)) != LOP_OK) return rc;
  const bool copy = h_out && !(P->flags & LOP_FLAG_NO_D2H);
  void* const direct = copy ? direct_host_target(P, P->sched == ChainSched::kWhole ? P->t.whole() : 0, h_out, true) : nullptr;
  rc = (P->flags & LOP_FLAG_GRAPH) && !timing && !enqueued_by_every_call(P, user != nullptr)
           ? launch_graph_merged(P, lane, d_in, d_out, direct, s)
           : enqueue_chain_merged(P, L, d_in, d_out, direct, s, user != nullptr);
  if (rc != LOP_OK) return rc;
  if ((rc = stamp(P->ev_c1)) != LOP_OK || (rc = stamp(P->ev_d0)) != LOP_OK) return rc;
  if (copy && !direct) {
    // (behind the graph, not a node of it: as a node of every lane's graph it held up the other
    // lanes' graphs, 198 against 161 us on a batch of two through the inverted-residual chain)
    rc = enqueue_band_copy(P, P->t.whole(), d_out, h_out, s);
    if (rc != LOP_OK) return rc;
  }
  if ((rc = stamp(P->ev_d1)) != LOP_OK) return rc;
  if (timing) LOP_HIP(hipEventRecord(P->ev_t1, s));
  return leave_lane(L);
}

// Copy-lane schedule of one band: its kernels on compute stream `cs` (as a graph of their own
// when graphs are on), its copy on the copy lane behind the band's "kernels finished" event.
int enqueue_band_with_copy_lane(lop_plan_t* P, int band, const void* d_in, void* d_out,
                                void* h_out, hipStream_t cs) {
  hipStream_t ds = P->lanes.back().stream;
  int rc;
  if (P->flags & LOP_FLAG_GRAPH) {
    rc = launch_graph(P, d_in, d_out, nullptr, cs, P->lane_index(band), band);
  } else {
    if (P->copied_valid[band]) {  // these rows of d_out may still be on their way to the host
      LOP_HIP(hipStreamWaitEvent(cs, P->ev_copied[band], 0));
      P->copied_valid[band] = 0;
    }
    rc = enqueue_band_kernels(P, band, d_in, d_out, cs);
  }
  if (rc != LOP_OK) return rc;
  LOP_HIP(hipEventRecord(P->ev_done[band], cs));
  LOP_HIP(hipStreamWaitEvent(ds, P->ev_done[band], 0));
  rc = enqueue_band_copy(P, band, d_out, h_out, ds);
  if (rc != LOP_OK) return rc;
  LOP_HIP(hipEventRecord(P->ev_copied[band], ds));
  P->copied_valid[band] = 1;
  return LOP_OK;
}

}  // namespace

extern "C" {

int lop_plan(const lop_layer_t* layers, int n_layers, const lop_tensor_desc_t* in, int n_bands,
             unsigned flags, lop_plan_t** out_plan) {
  if (!out_plan) return LOP_ERR_INVALID_ARG;
  *out_plan = nullptr;
  lop_plan_t* P = new (std::nothrow) lop_plan_t;
  if (!P) return LOP_ERR_OOM;
  int rc = lop::build_tables(layers, n_layers, in, n_bands, (flags & LOP_FLAG_REUSE) != 0, P->t);
  if (rc != LOP_OK) { delete P; return rc; }
  P->flags = flags;
  P->k_pad.assign((size_t)n_layers, 0);  // padded reduction length of every dense conv
  P->has_wd.assign((size_t)n_layers, 0);
  P->has_wd16.assign((size_t)n_layers, 0);
  P->has_w3.assign((size_t)n_layers, 0);
  P->has_wstem.assign((size_t)n_layers, 0);
  const int ke = 16 / (int)P->t.esz();
  for (int l = 0; l < n_layers; ++l) {
    const lop_layer_t& d = P->t.layers[l].d;
    if (d.op != LOP_CONV2D) continue;
    P->k_pad[l] = lop::conv_k_pad(d.c_in, d.kh, d.kw, in->dtype);
    P->has_wd[l] = d.c_in % ke == 0 && d.c_out % ke == 0;
    P->has_wd16[l] = P->has_wd[l] && P->k_pad[l] % (4 * ke) == 0;
    P->has_w3[l] = in->dtype == LOP_F32 && P->has_wd[l] && lop::split_shape(d.c_in, d.kh, d.kw, d.sh, d.sw, std::max(d.dh, d.dw));
    P->has_wstem[l] = lop::stem_shape_applies(d.c_in, d.c_out, d.kh, d.kw, d.sw, d.dh, d.dw,
                                              d.residual_from != LOP_NO_RESIDUAL);
  }
  find_fused_groups(P, false, &P->fuse_band);
  find_fused_groups(P, true, &P->fuse_chain);
  if (flags & LOP_FLAG_BATCH_BANDS) {
    if (flags & LOP_FLAG_REUSE) { delete P; return LOP_ERR_INVALID_ARG; }
    if (!all_launches_batchable(P)) { delete P; return LOP_ERR_UNSUPPORTED; }
    P->batched = true;
  }
  size_scratch(P);
  if (!(flags & LOP_FLAG_PLAN_ONLY)) {
    rc = setup_device(P);
    if (rc != LOP_OK) { lop_plan_destroy(P); return rc; }
    P->ready = true;
  }
  *out_plan = P;
  return LOP_OK;
}

int lop_plan_rowwise(const lop_rowwise_t* layers, int n_layers, int m, int k, int dtype, int n_bands,
                     unsigned flags, lop_plan_t** out_plan) {
  if (!out_plan) return LOP_ERR_INVALID_ARG;
  *out_plan = nullptr;
  if (!layers || n_layers < 1 || m < 1 || k < 1) return LOP_ERR_INVALID_ARG;
  // a matrix row is a pixel of an m x 1 image with k channels; the product is a 1x1 conv
  std::vector<lop_layer_t> conv((size_t)n_layers);
  for (int l = 0; l < n_layers; ++l) {
    const lop_rowwise_t& r = layers[l];
    lop_layer_t& c = conv[l];
    c.op = LOP_CONV2D;
    c.c_in = r.k; c.c_out = r.n;
    c.kh = c.kw = c.sh = c.sw = c.dh = c.dw = 1;
    c.ph = c.pw = 0;
    c.act = r.act;
    c.input_from = r.input_from;
    c.residual_from = r.residual_from;
    c.weight = r.weight;
    c.bias = r.bias;
  }
  const lop_tensor_desc_t in{1, k, m, 1, dtype};
  return lop_plan(conv.data(), n_layers, &in, n_bands, flags, out_plan);
}

void lop_plan_destroy(lop_plan_t* P) {
  if (!P) return;
  if (P->ready || P->device >= 0) {
    // Everything below belongs to the plan's device, and work that uses the plan's memory may
    // sit on streams the plan does not own (a caller's compute or copy stream, which may not
    // exist any more, so it is not touched through its handle): wait for the whole device.
    int cur = -1;
    if (hipGetDevice(&cur) == hipSuccess && cur != P->device && P->device >= 0) (void)hipSetDevice(P->device);
    (void)hipDeviceSynchronize();
  }
  for (void* w : P->d_w) if (w) (void)lop::dev_free(w);
  for (void* w : P->d_wd) if (w) (void)lop::dev_free(w);
  for (void* w : P->d_wd16) if (w) (void)lop::dev_free(w);
  for (void* w : P->d_wstem) if (w) (void)lop::dev_free(w);
  for (float* b : P->d_bias) if (b) (void)lop::dev_free(b);
  for (auto* v : {&P->ev_done, &P->ev_copied, &P->ev_c0, &P->ev_c1, &P->ev_d0, &P->ev_d1})
    for (hipEvent_t e : *v) if (e) (void)hipEventDestroy(e);
  for (auto& g : P->graphs) (void)hipGraphExecDestroy(g.exec);
  for (hipEvent_t e : {P->ev_fork, P->ev_t0, P->ev_t1, P->ev_copy_tail}) if (e) (void)hipEventDestroy(e);
  for (Lane& L : P->lanes) {
    if (L.arena) (void)lop::dev_free(L.arena);
    if (L.conv_ws) (void)lop::dev_free(L.conv_ws);
    if (L.ev_join) (void)hipEventDestroy(L.ev_join);
    if (L.stream) (void)hipStreamDestroy(L.stream);
    if (L.copy) (void)hipStreamDestroy(L.copy);
  }
  if (P->s_main) (void)hipStreamDestroy(P->s_main);
  if (P->s_copy) (void)hipStreamDestroy(P->s_copy);
  delete P;
}

int lop_plan_out_desc(const lop_plan_t* P, lop_tensor_desc_t* out) {
  if (!P || !out) return LOP_ERR_INVALID_ARG;
  return lop_plan_layer_desc(P, P->t.n_layers() - 1, out);
}

int lop_plan_layer_desc(const lop_plan_t* P, int layer, lop_tensor_desc_t* out) {
  if (!P || !out) return LOP_ERR_INVALID_ARG;
  if (layer < 0 || layer >= P->t.n_layers()) return LOP_ERR_BAND_RANGE;
  const lop::LayerInfo& L = P->t.layers[layer];
  *out = {L.n, L.d.c_out, L.h_out, L.w_out, P->t.in.dtype};
  return LOP_OK;
}

int lop_plan_n_bands(const lop_plan_t* P) { return P ? P->t.n_bands : LOP_ERR_INVALID_ARG; }
int lop_plan_n_layers(const lop_plan_t* P) { return P ? P->t.n_layers() : LOP_ERR_INVALID_ARG; }

int lop_plan_band_layer_rows(const lop_plan_t* P, int band, int layer, lop_rows_t* rows) {
  if (!P || !rows) return LOP_ERR_INVALID_ARG;
  if (band < 0 || band >= P->t.n_bands || layer < -1 || layer >= P->t.n_layers())
    return LOP_ERR_BAND_RANGE;
  lop_rows_t r = P->t.bands[band].need[layer + 1];
  if (r.hi <= r.lo) r = {0, 0};
  *rows = r;
  return LOP_OK;
}

int lop_plan_band_out_rows(const lop_plan_t* P, int band, lop_rows_t* rows) {
  if (!P || !rows) return LOP_ERR_INVALID_ARG;
  if (band < 0 || band >= P->t.n_bands) return LOP_ERR_BAND_RANGE;
  *rows = P->t.bands[band].need[P->t.n_layers()];  // split intervals keep lo == hi when empty
  return LOP_OK;
}

int lop_plan_band_compute_rows(const lop_plan_t* P, int band, int layer, lop_rows_t* rows) {
  if (!P || !rows) return LOP_ERR_INVALID_ARG;
  if (band < 0 || band >= P->t.n_bands || layer < 0 || layer >= P->t.n_layers())
    return LOP_ERR_BAND_RANGE;
  lop_rows_t r = P->t.bands[band].compute[layer];
  if (r.hi <= r.lo) r = {0, 0};
  *rows = r;
  return LOP_OK;
}

int lop_plan_band_in_rows(const lop_plan_t* P, int band, lop_rows_t* rows) {
  return lop_plan_band_layer_rows(P, band, -1, rows);
}

int lop_plan_stats(const lop_plan_t* P, double* useful, double* executed, size_t* scratch) {
  if (!P) return LOP_ERR_INVALID_ARG;
  double u = 0, e = 0;
  for (int l = 0; l < P->t.n_layers(); ++l) {
    u += P->t.layer_flop(l, P->t.layers[l].h_out);
    for (int b = 0; b < P->t.n_bands; ++b) {
      double f = 0.0, by = 0.0;
      if (P->flags & LOP_FLAG_PLAN_ONLY) {  // no kernels are chosen, so no launches are fused
        const lop_rows_t r = P->t.bands[b].compute[l];
        if (r.hi > r.lo) f = P->t.layer_flop(l, r.hi - r.lo);
      } else {
        launch_work(P, b, l, &f, &by);
      }
      e += f;
    }
  }
  if (useful) *useful = u;
  if (executed) *executed = e;
  if (scratch) *scratch = align_up(P->arena_bytes, 256) + P->conv_ws_bytes;
  return LOP_OK;
}

int lop_plan_layer_work(const lop_plan_t* P, int band, int layer, double* flop, double* bytes) {
  if (!P) return LOP_ERR_INVALID_ARG;
  if (band < 0 || band >= P->t.n_bands || layer < 0 || layer >= P->t.n_layers())
    return LOP_ERR_BAND_RANGE;
  double f = 0.0, by = 0.0;
  if (P->flags & LOP_FLAG_PLAN_ONLY) {  // no kernels are chosen, so no launches are fused
    const lop_rows_t r = P->t.bands[band].compute[layer];
    f = r.hi > r.lo ? P->t.layer_flop(layer, r.hi - r.lo) : 0.0;
    by = P->t.layer_bytes(band, layer);
  } else {
    launch_work(P, band, layer, &f, &by);
  }
  if (flop) *flop = f;
  if (bytes) *bytes = by;
  return LOP_OK;
}

// The kernels move 16-byte vectors: tensors start on a 16-byte boundary.
static bool misaligned(const void* p) { return ((uintptr_t)p & 15u) != 0; }

int lop_run_band(lop_plan_t* P, int band, const void* d_in, void* d_out, void* h_out,
                 void* compute_stream, void* copy_stream) {
  if (!P || !d_in || !d_out) return LOP_ERR_INVALID_ARG;
  if (misaligned(d_in) || misaligned(d_out) || misaligned(h_out)) return LOP_ERR_INVALID_ARG;
  if (band < 0 || band >= P->t.n_bands) return LOP_ERR_BAND_RANGE;
  if (!P->ready) return LOP_ERR_NOT_READY;
  if (band_empty(P, band)) return LOP_OK;
  if (h_out && !(P->flags & LOP_FLAG_NO_D2H) && !device_view_of_host(P, h_out)) return LOP_ERR_INVALID_ARG;
  hipStream_t cs = compute_stream ? (hipStream_t)compute_stream : P->lane_of(band).stream;
  hipStream_t ds = copy_stream ? (hipStream_t)copy_stream : P->s_copy;
  if (compute_stream) P->last_user_stream = cs;
  Lane& L = P->lane_of(band);
  int rc = take_lane(L, cs);
  if (rc == LOP_OK) rc = enqueue_band(P, band, d_in, d_out, h_out, cs, ds, false);
  return rc == LOP_OK ? leave_lane(L) : rc;
}

int lop_run_chain(lop_plan_t* P, const void* d_in, void* d_out, void* h_out, void* compute_stream,
                  lop_timing_t* timing) {
  if (!P || !d_in || !d_out) return LOP_ERR_INVALID_ARG;
  if (misaligned(d_in) || misaligned(d_out) || misaligned(h_out)) return LOP_ERR_INVALID_ARG;
  if (!P->ready) return LOP_ERR_NOT_READY;
  hipStream_t ms = compute_stream ? (hipStream_t)compute_stream : P->s_main;
  if (compute_stream) P->last_user_stream = ms;
  const int nb = P->t.n_bands;
  const bool copy = h_out && !(P->flags & LOP_FLAG_NO_D2H);
  if (copy && !device_view_of_host(P, h_out)) return LOP_ERR_INVALID_ARG;  // not pinned host memory
  if (timing) {
    int rc = ensure_timing_events(P);
    if (rc != LOP_OK) return rc;
    rc = lop_synchronize(P);
    if (rc != LOP_OK) return rc;
  }
  const auto t0 = std::chrono::steady_clock::now();
  // (with timing the bands of a plan that did not ask for batched launches run one by one, so
  // that each has a start and an end of its own)
  const bool merged = P->sched != ChainSched::kPerBand && (!timing || P->batched);
  // (one graph of all bands runs on `ms` itself, with every lane's scratch)
  const bool lanes_in_graph = !merged && !P->t.reuse && (P->flags & LOP_FLAG_GRAPH) && !timing &&
                              (compute_stream || P->n_lanes() == 1) && !(P->copy_lane && copy && !compute_stream);
  hipEvent_t waited = nullptr;
  if (!merged)
    for (Lane& L : P->lanes) {   // a band or a chain on a caller's stream may still use a lane's scratch
      int rc = lanes_in_graph ? take_lane(L, ms, &waited) : take_lane(L, L.stream);
      if (rc != LOP_OK) return rc;
    }
  if (P->copy_lane && copy && !compute_stream && !timing) {
    // Compute lanes run free, as below; every band's copy goes to the copy lane.
    for (int b = 0; b < nb; ++b) {
      if (band_empty(P, b)) continue;
      int rc = enqueue_band_with_copy_lane(P, b, d_in, d_out, h_out, P->lane_of(b).stream);
      if (rc != LOP_OK) return rc;
    }
    return LOP_OK;
  }
  // (on a caller's stream, bands in a row or one lane's)
  const ChainAlone scope(P, compute_stream && !merged && (P->t.reuse || P->n_lanes() == 1));
  if (merged) {
    int rc = run_merged(P, d_in, d_out, h_out, compute_stream ? ms : nullptr, timing != nullptr);
    if (rc != LOP_OK) return rc;
  } else if (P->t.reuse) {
    // the whole chain runs on one lane; chains of consecutive calls rotate over the lanes
    // and overlap unless the caller's stream orders them
    P->cur_lane = P->next_lane;
    P->next_lane = (P->next_lane + 1) % P->n_lanes();
    Lane& L = P->lanes[P->cur_lane];
    if (compute_stream) {
      LOP_HIP(hipEventRecord(P->ev_fork, ms));
      LOP_HIP(hipStreamWaitEvent(L.stream, P->ev_fork, 0));
    }
    if (timing) LOP_HIP(hipEventRecord(P->ev_t0, L.stream));
    int rc = ((P->flags & LOP_FLAG_GRAPH) && !timing)
                 ? launch_graph(P, d_in, d_out, h_out, L.stream)
                 : enqueue_chain_reuse(P, d_in, d_out, h_out, timing != nullptr, false);
    if (rc != LOP_OK) return rc;
    if (timing) LOP_HIP(hipEventRecord(P->ev_t1, L.stream));
    if (compute_stream) {
      LOP_HIP(hipEventRecord(L.ev_join, L.stream));
      LOP_HIP(hipStreamWaitEvent(ms, L.ev_join, 0));
    }
  } else {
    if (!compute_stream && !timing && P->n_lanes() > 1) {
      // No stream of the caller's to order against: every lane takes its bands of this chain
      // behind whatever it still has of earlier chains and nothing joins them, so the lanes
      // drift apart by as much as their bands differ in work and consecutive chains overlap
      // (band b of the next chain starts while slower bands of this one still run). The
      // chain is complete after lop_synchronize.
      for (int k = 0; k < P->n_lanes(); ++k) {
        int rc = (P->flags & LOP_FLAG_GRAPH) ? launch_graph(P, d_in, d_out, h_out, P->lanes[k].stream, k)
                                             : enqueue_lane(P, k, d_in, d_out, h_out, false);
        if (rc != LOP_OK) return rc;
      }
      return LOP_OK;
    }
    if (lanes_in_graph) {
      int rc = launch_graph(P, d_in, d_out, h_out, ms);
      const int left = leave_lanes(P);   // (also after an error: a capture may have used the lanes' events)
      return rc == LOP_OK ? left : rc;
    }
    if (timing) LOP_HIP(hipEventRecord(P->ev_t0, ms));
    int rc = enqueue_chain(P, d_in, d_out, h_out, ms, timing != nullptr, false);
    if (rc != LOP_OK) return rc;
    if (timing) LOP_HIP(hipEventRecord(P->ev_t1, ms));
  }
  if (!timing) return LOP_OK;
  int rc = lop_synchronize(P);
  if (rc != LOP_OK) return rc;
  const auto t1 = std::chrono::steady_clock::now();
  std::memset(timing, 0, sizeof(*timing));
  timing->n_bands = nb;
  timing->wall_ms = std::chrono::duration<float, std::milli>(t1 - t0).count();
  for (int b = 0; b < nb; ++b) {
    if (band_empty(P, b)) continue;
    LOP_HIP(hipEventElapsedTime(&timing->band_compute_ms[b], P->ev_c0[b], P->ev_c1[b]));
    if (copy) {
      LOP_HIP(hipEventElapsedTime(&timing->band_copy_ms[b], P->ev_d0[b], P->ev_d1[b]));
      timing->copy_ms += timing->band_copy_ms[b];
    }
    LOP_HIP(hipEventElapsedTime(&timing->band_ready_ms[b], P->ev_t0, copy ? P->ev_d1[b] : P->ev_c1[b]));
  }
  LOP_HIP(hipEventElapsedTime(&timing->compute_ms, P->ev_t0, P->ev_t1));
  return LOP_OK;
}

int lop_run_chain_static(lop_plan_t* P, const void* d_in, void* d_out, void* stream) {
  if (!P || !d_in || !d_out) return LOP_ERR_INVALID_ARG;
  if (misaligned(d_in) || misaligned(d_out)) return LOP_ERR_INVALID_ARG;
  if (!P->ready) return LOP_ERR_NOT_READY;
  const size_t arena = align_up(P->arena_bytes, 256);
  if (arena + P->conv_ws_bytes > (size_t)LOP_STATIC_SCRATCH_BYTES) return LOP_ERR_TOO_LARGE;
  unsigned char* const base = (unsigned char*)static_scratch_of(P->device);
  if (!base) return LOP_ERR_NOT_READY;
  // Nothing in the array has to start at zero: a band's slabs are written by the layer that
  // produces them before any layer reads them, and a launch's partial sums by its slices
  // before its finish kernel adds them, so the contents left by the last call do not matter.
  ChainScratch scratch(P, base, P->conv_ws_bytes ? base + arena : nullptr, true);
  if (P->sched != ChainSched::kPerBand) return enqueue_merged_kernels(P, d_in, d_out, (hipStream_t)stream, nullptr);
  int rc = LOP_OK;
  for (int b = 0; b < P->t.n_bands && rc == LOP_OK; ++b)
    if (!band_empty(P, b)) rc = enqueue_band_kernels(P, b, d_in, d_out, (hipStream_t)stream);
  return rc;
}

int lop_synchronize(lop_plan_t* P) {
  if (!P) return LOP_ERR_INVALID_ARG;
  if (!P->ready) return LOP_ERR_NOT_READY;
  if (P->last_user_stream) LOP_HIP(hipStreamSynchronize(P->last_user_stream));
  for (int b = 0; b < P->t.n_bands; ++b)   // copies of single bands, on streams of the caller's
    if (P->copied_valid[b]) LOP_HIP(hipEventSynchronize(P->ev_copied[b]));
  for (Lane& L : P->lanes) {
    if (L.user) LOP_HIP(hipEventSynchronize(L.left));
    LOP_HIP(hipStreamSynchronize(L.stream));
    LOP_HIP(hipStreamSynchronize(L.copy));
  }
  LOP_HIP(hipStreamSynchronize(P->s_main));
  LOP_HIP(hipStreamSynchronize(P->s_copy));
  return LOP_OK;
}

int lop_time_layer(lop_plan_t* P, int band, int layer, const void* d_in, void* d_out, int iters,
                   float* ms_per_launch) {
  if (!P || !d_in || !d_out || !ms_per_launch || iters < 1) return LOP_ERR_INVALID_ARG;
  if (misaligned(d_in) || misaligned(d_out)) return LOP_ERR_INVALID_ARG;
  if (band < 0 || band >= P->t.n_bands || layer < 0 || layer >= P->t.n_layers())
    return LOP_ERR_BAND_RANGE;
  if (!P->ready) return LOP_ERR_NOT_READY;
  *ms_per_launch = 0.f;
  const lop_rows_t r = launch_rows(P, band_fusion(P), band, layer);
  if (r.hi <= r.lo) return LOP_OK;
  int rc = ensure_timing_events(P);
  if (rc == LOP_OK) rc = lop_synchronize(P);   // (a chain in flight may be using the lane's scratch)
  if (rc != LOP_OK) return rc;
  hipStream_t cs = P->s_main;
  LOP_HIP(launch_layer(P, band_fusion(P), band, layer, d_in, d_out, cs));  // warm-up
  LOP_HIP(hipEventRecord(P->ev_c0[0], cs));
  for (int i = 0; i < iters; ++i) LOP_HIP(launch_layer(P, band_fusion(P), band, layer, d_in, d_out, cs));
  LOP_HIP(hipEventRecord(P->ev_c1[0], cs));
  LOP_HIP(hipStreamSynchronize(cs));
  float ms = 0.f;
  LOP_HIP(hipEventElapsedTime(&ms, P->ev_c0[0], P->ev_c1[0]));
  *ms_per_launch = ms / iters;
  return LOP_OK;
}

int lop_plan_layer_kernel(const lop_plan_t* P, int band, int layer, char* name, size_t size,
                          int* k_slices) {
  if (!P || !name || size == 0) return LOP_ERR_INVALID_ARG;
  if (band < 0 || band >= P->t.n_bands || layer < 0 || layer >= P->t.n_layers())
    return LOP_ERR_BAND_RANGE;
  name[0] = 0;
  int slices = 0;
  // (a plan-only plan has uploaded no weights, and which kernel takes a layer depends on the
  // packings that exist: it names none rather than a kernel the ready plan would not launch)
  if (P->flags & LOP_FLAG_PLAN_ONLY) {
  } else if (P->batched) {   // one launch per layer for all bands: named at the first band that takes part
    if (batched_owner(P, layer) == band) slices = describe_layer_batched(P, layer, name, size);
  } else {
    slices = describe_layer_launch(P, band, layer, name, size);
  }
  if (k_slices) *k_slices = slices;
  return LOP_OK;
}

int lop_profile_chain(lop_plan_t* P, const void* d_in, void* d_out, int iters, float* layer_ms,
                      float* finish_ms) {
  if (!P || !d_in || !d_out || !layer_ms || iters < 1) return LOP_ERR_INVALID_ARG;
  if (misaligned(d_in) || misaligned(d_out)) return LOP_ERR_INVALID_ARG;
  if (!P->ready) return LOP_ERR_NOT_READY;
  const int nb = P->t.n_bands, nl = P->t.n_layers();
  int rc = lop_synchronize(P);
  if (rc != LOP_OK) return rc;
  hipStream_t cs = P->s_main;
  // (start, stop) of the operator's kernel and of its finish kernel, attached to the
  // dispatches themselves
  std::vector<hipEvent_t> ev((size_t)nb * nl * 4, nullptr);
  std::vector<int> used((size_t)nb * nl, 0);
  auto run = [&]() -> int {
    for (auto& e : ev) LOP_HIP(hipEventCreate(&e));
    for (int i = 0; i < nb * nl; ++i) {
      layer_ms[i] = 0.f;
      if (finish_ms) finish_ms[i] = 0.f;
    }
    for (int it = 0; it < iters; ++it) {
      for (int b = 0; b < nb; ++b)
        for (int l = 0; l < nl; ++l) {
          const lop_rows_t r = launch_rows(P, band_fusion(P), b, l);
          if (r.hi <= r.lo) continue;
          if (P->batched && batched_owner(P, l) != b) continue;  // (timed with the band that owns the launch)
          const size_t i = ((size_t)b * nl + l) * 4;
          lop::KernelEvents ke;
          ke.start[0] = ev[i]; ke.stop[0] = ev[i + 1];
          ke.start[1] = ev[i + 2]; ke.stop[1] = ev[i + 3];
          const ChainPass pass(P, 0, P->batched ? P->images : 0);
          if (P->batched) LOP_HIP(launch_layer_batched(P, l, 0, nb, d_in, d_out, cs, &ke, nullptr));
          else LOP_HIP(launch_layer(P, P->fuse_band, b, l, d_in, d_out, cs, &ke));
          used[b * nl + l] = ke.n;
        }
      LOP_HIP(hipStreamSynchronize(cs));
      for (int b = 0; b < nb; ++b)
        for (int l = 0; l < nl; ++l) {
          const size_t i = ((size_t)b * nl + l) * 4;
          float ms = 0.f, fin = 0.f;
          if (used[b * nl + l] >= 1) LOP_HIP(hipEventElapsedTime(&ms, ev[i], ev[i + 1]));
          if (used[b * nl + l] >= 2) LOP_HIP(hipEventElapsedTime(&fin, ev[i + 2], ev[i + 3]));
          layer_ms[b * nl + l] += ms / iters;
          if (finish_ms) finish_ms[b * nl + l] += fin / iters;
        }
    }
    return LOP_OK;
  };
  rc = run();
  for (hipEvent_t e : ev) if (e) (void)hipEventDestroy(e);
  return rc;
}

int lop_copy_chain(lop_plan_t* P, const void* d_out, void* h_out) {
  if (!P || !d_out || !h_out) return LOP_ERR_INVALID_ARG;
  if (misaligned(d_out) || misaligned(h_out)) return LOP_ERR_INVALID_ARG;
  if (!P->ready) return LOP_ERR_NOT_READY;
  if (!device_view_of_host(P, h_out)) return LOP_ERR_INVALID_ARG;
  for (int b = 0; b < P->t.n_bands; ++b) {
    int rc = enqueue_band_copy(P, b, d_out, h_out, P->s_copy);
    if (rc != LOP_OK) return rc;
  }
  return LOP_OK;
}

const char* lop_strerror(int code) {
  switch (code) {
    case LOP_OK: return "ok";
    case LOP_ERR_INVALID_ARG: return "invalid argument";
    case LOP_ERR_UNSUPPORTED: return "unsupported operator, type or parameter";
    case LOP_ERR_SHAPE: return "shape mismatch";
    case LOP_ERR_BAND_RANGE: return "band or layer index out of range";
    case LOP_ERR_OOM: return "out of memory";
    case LOP_ERR_HIP: return "HIP runtime error";
    case LOP_ERR_NOT_READY: return "plan holds no device state (plan-only)";
    case LOP_ERR_TOO_LARGE: return "the plan needs more scratch than the static array holds";
    default: return "unknown error";
  }
}

int lop_last_hip_error(void) { return g_last_hip; }

}  // extern "C"
