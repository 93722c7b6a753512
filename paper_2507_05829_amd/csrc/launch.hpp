// One place where kernels are launched, so that a launch can carry the events that time it.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstddef>

#include "kernels.hpp"

namespace lop {

// Launches `kernel`; with `ev` the next free (start, stop) pair is attached to the dispatch
// itself, so their difference is the kernel's own duration as a profiler reports it (an event
// recorded before and after a launch also spans the gaps between dispatches).
template <typename... KArgs, typename... Args>
inline hipError_t launch_kernel(void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t s,
                                KernelEvents* ev, Args... args) {
  if (ev && ev->n < KernelEvents::kMax) {
    const int i = ev->n++;
    hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev->start[i], ev->stop[i], 0,
                          static_cast<KArgs>(args)...);
  } else {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, static_cast<KArgs>(args)...);
  }
  return hipGetLastError();
}

// Several launches of one operator - the bands of a chain at one layer - as one grid (the
// operation batching of Sec. IV-D: the local operations a device holds of one operator go
// into one kernel call). Band b owns the blocks first[b] .. first[b + 1] of the grid's x
// dimension and has its own parameters; y and z extents are the same for every band.
constexpr int kMaxBatch = 16;
template <typename P>
struct Batch {
  int n;
  int first[kMaxBatch + 1];
  P p[kMaxBatch];
};
template <typename P>
__device__ __forceinline__ int batch_find(const Batch<P>& t, int bx) {
  int b = 0;
  while (b + 1 < t.n && bx >= t.first[b + 1]) ++b;
  return b;
}

// Reads a word of every 64-byte line of the kernel's arguments from `offset` on, all at once. Left to itself a kernel loads a
// parameter shortly before it needs it, line after line of memory that no cache holds yet when a launch starts (a chain of
// 13 launches over eight bands, alone: 246 -> 239 us).
template <int BYTES>
__device__ __forceinline__ void touch_arguments(int offset = 0) {
  const auto* const at = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() + offset;
  auto word = [&](int i) __attribute__((always_inline)) { return *(const __attribute__((address_space(4))) int*)(at + (i < BYTES - 4 ? i : BYTES - 4)); };
  asm volatile("" ::"s"(word(0)), "s"(word(64)), "s"(word(128)), "s"(word(192)), "s"(word(256)));
}
template <typename P>
__device__ __forceinline__ int find_band(const Batch<P>& t, int bx) {
  const int b = batch_find(t, bx);
  touch_arguments<sizeof(P)>((int)offsetof(Batch<P>, p) + b * (int)sizeof(P));
  return b;
}

// One band: the kernel itself; several bands of the layer: its _bands form on a grid whose x
// extent is the sum of the bands' (gx: blocks of x per band).
template <typename P>
inline hipError_t launch_group(void (*single)(const P), void (*bands)(const Batch<P>), const P* ps, int n,
                               const unsigned* gx, unsigned gy, unsigned gz, dim3 block, hipStream_t s,
                               KernelEvents* ev) {
  if (n < 1 || n > kMaxBatch || gy > 65535 || gz > 65535) return hipErrorInvalidValue;
  if (n == 1) return launch_kernel(single, dim3(gx[0], gy, gz), block, s, ev, ps[0]);
  Batch<P> t;
  t.n = n;
  unsigned long at = 0;
  for (int b = 0; b < kMaxBatch; ++b) {
    t.first[b] = (int)at;
    t.p[b] = ps[b < n ? b : n - 1];
    if (b < n) at += gx[b];
  }
  t.first[kMaxBatch] = (int)at;
  if (at == 0 || at > 0x7fffffffUL) return hipErrorInvalidValue;
  return launch_kernel(bands, dim3((unsigned)at, gy, gz), block, s, ev, t);
}

}  // namespace lop
