// Waits of a ring of direct global -> LDS loads: __syncthreads() would wait for every outstanding load and empty the ring.
#pragma once
#include <hip/hip_runtime.h>

namespace ldsring {

// waits until at most N of this wavefront's vector-memory loads are outstanding (they complete in order)
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// waits until at most `left` (<= LEFT) stages of OPS loads are outstanding
template <int OPS, int LEFT>
__device__ __forceinline__ void wait_stages(int left) {
  if constexpr (LEFT == 0) wait_loads<0>();
  else {
    if (left >= LEFT) wait_loads<LEFT * OPS>();
    else wait_stages<OPS, LEFT - 1>(left);
  }
}

// this wavefront's LDS reads are done
__device__ __forceinline__ void wait_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// barrier behind the LDS reads that leaves vector-memory loads in flight
__device__ __forceinline__ void barrier_keep_loads() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace ldsring
