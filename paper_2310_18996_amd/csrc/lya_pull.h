// Work queue of the kernels that take lines wave by wave.  Additions to one cache
// line are served one after the other, 11.5 ns each (measured; 1.0 ns over 16
// lines): 50,000 lines in pulls of four took 140 us for the pulls alone, and a
// kernel whose waves all start at once waited 35-45 us for its first ones.  So
// the queue is 16 counters, each in its own line: counter k hands out the chunks
// 16 i + k, and a wave whose counter has run out goes on with another that has not.
#pragma once

#include "lya_internal.h"

namespace lya {

// A kernel's first argument, to be read where it is used: arguments that the
// compiler loads at the kernel's start stay in scalar registers all along, and
// where they do not fit each use takes a lane read.
template <typename A>
using KernArg = const __attribute__((address_space(4))) A;
template <typename A>
__device__ __forceinline__ KernArg<A>* kernarg_here() {
  auto* p = (KernArg<A>*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// The chunks of a wave of a kernel whose argument is an A with queue, chunk,
// chunks, in blocks of WAVES waves: c = first(), while c < chunks: ask() before
// the chunk's last line, c = next().  A grid with a wave for every chunk takes
// them by number, without the counters; else even the first comes from them, so
// that blocks which start late (a grid beyond what the device holds at once)
// find only what is left.  What a wave keeps meanwhile is one vector register.
template <typename A, int WAVES>
struct LinePull {
  uint32_t way;     // lane 0: the pull on its way; lane 1: counter; lane 2: counters not known to be empty

  __device__ __forceinline__ static bool one_each(int64_t n) { return n <= static_cast<int64_t>(gridDim.x) * WAVES; }
  __device__ __forceinline__ int64_t first(int lane) {
    if (one_each(kernarg_here<A>()->chunks))
      return __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x) * WAVES + static_cast<int>(threadIdx.x >> 6));
    way = lane == 1 ? blockIdx.x % kPullCounters : (1u << kPullCounters) - 1u;
    ask(lane);
    return next(lane);
  }
  __device__ __forceinline__ void ask(int lane) {
    const auto* a = kernarg_here<A>();
    if (one_each(a->chunks)) return;
    const uint32_t k = __builtin_amdgcn_readlane(way, 1);
    if (lane == 0) way = atomicAdd(a->queue + k * kPullStride, 1u);
  }
  __device__ __forceinline__ int64_t next(int lane) {
    const auto* a = kernarg_here<A>();
    const int64_t n = a->chunks;
    if (one_each(n)) return n;
    while (true) {
      const uint32_t k = __builtin_amdgcn_readlane(way, 1);
      const int64_t c = static_cast<int64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(way))) * kPullCounters + k;
      if (c < n) return c;
      const uint32_t open = __builtin_amdgcn_readlane(way, 2) & ~(1u << k);   // never asked again, so this ends
      // what the other counters have handed out (a value read too early only
      // costs a pull in vain)
      bool left = false;
      if (lane < kPullCounters && (open >> lane & 1u)) {
        const uint32_t v = __hip_atomic_load(a->queue + lane * kPullStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        left = static_cast<int64_t>(v) * kPullCounters + lane < n;
      }
      const uint32_t some = static_cast<uint32_t>(__ballot(left));
      if (some == 0u) return n;
      const uint32_t up = some >> k << k;   // the next one up, around the end
      way = lane == 1 ? static_cast<uint32_t>(__builtin_ctz(up ? up : some)) : open;
      ask(lane);
    }
  }
};

}  // namespace lya
