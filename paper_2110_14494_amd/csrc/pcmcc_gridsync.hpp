// Grid-wide barrier of the persistent kernels, with a completion step.
//
// A persistent step kernel needs, at every barrier, a few numbers that the
// phase before it left in device counters (how many newborns were queued,
// how many holes there are, whether something overflowed).  Read by every
// wave after the barrier they cost far more than the barrier itself: all
// waves of the grid load one address at device scope, which is served one
// wave after the other (4096 waves: 10 to 32 us for each word on a grid of
// 512 blocks of 8 waves), and a commit by one block needs a second barrier.
// Here the last block to arrive runs a completion function on its own while
// the others wait, and publishes what it returns in the words the others
// are waiting for: one barrier costs 5.6 us over 256 blocks and 9.5 us over
// 512 (of 256 or 512 threads, one after the other without work between them),
// the numbers included.
//
// Arrivals are counted in kBarGroups counters on cache lines of their own
// (a same-address atomic takes about 13 ns on this device, 6.6 us for 512
// blocks on one counter), the last of a group arrives at the root.  The
// result words carry the barrier's number in their upper half, so a waiting
// wave sees from the word itself that it is the new one, and are written
// once per kBarCopies, so that the waiting blocks poll different lines.
//
// Every block of the grid must be resident (cooperative launch), every
// thread of every block must call, and the GridBar must be zero when the
// kernel starts (`gen` starts at 0).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pcmcc {

constexpr unsigned kBarGroups = 16, kBarCopies = 8, kBarWords = 8;

struct alignas(128) BarLine {
  unsigned v;
};
struct alignas(128) BarWords {
  unsigned long long w[kBarWords];
};
struct GridBar {
  BarLine arrive[kBarGroups];
  BarLine root;
  BarWords pub[kBarCopies];
};

template <class T>
__device__ __forceinline__ T ld_relaxed(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void st_relaxed(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Barrier number ++gen: everything the grid wrote before it is visible to
// the completion function and to everyone after it.  complete(v) is called
// once, by one thread, with v[kBarWords] set to zero; s_pub (LDS,
// kBarWords words) holds v in every block on return, until the block's next
// barrier.
template <class Fn>
__device__ __forceinline__ void grid_barrier(GridBar* B, uint32_t& gen, uint32_t* s_pub, Fn&& complete) {
  // this wave's stores have left it before the block's thread 0 releases
  // them for the whole block
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
  ++gen;
  if (threadIdx.x < 64) {
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      const uint32_t grp = blockIdx.x % kBarGroups;
      const uint32_t members = (gridDim.x - grp + kBarGroups - 1) / kBarGroups;
      const uint32_t groups = gridDim.x < kBarGroups ? gridDim.x : kBarGroups;
      if (atomicAdd(&B->arrive[grp].v, 1u) + 1u == gen * members) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
        if (atomicAdd(&B->root.v, 1u) + 1u == gen * groups) {
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          uint32_t v[kBarWords] = {0};
          complete(v);
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
          for (unsigned c = 0; c < kBarCopies; ++c)
#pragma unroll
            for (unsigned q = 0; q < kBarWords; ++q)
              st_relaxed(&B->pub[c].w[q], ((unsigned long long)gen << 32) | v[q]);
        }
      }
    }
    const unsigned long long* src = &B->pub[blockIdx.x % kBarCopies].w[threadIdx.x % kBarWords];
    unsigned long long w;
    for (;;) {
      w = ld_relaxed(src);
      if (__ballot((uint32_t)(w >> 32) != gen) == 0) break;
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (threadIdx.x < kBarWords) s_pub[threadIdx.x] = (uint32_t)w;
  }
  __syncthreads();
}

// Sum of v over the wave, in every lane (data-parallel-primitive adds: no
// LDS round trips).
__device__ __forceinline__ uint32_t wave_sum_dpp(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, true);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, true);  // row_bcast:31
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

}  // namespace pcmcc
