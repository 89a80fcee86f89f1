// Cross-workgroup publication inside one launch (dataflow Cholesky, solves):
// agent-coherent loads and stores, bounded flag waits that raise an error
// word, and the flag store after a workgroup's data stores have drained.
// Header-only: included by each kernel file that publishes or consumes.
#pragma once
#include "common.h"

namespace pdk {

// The thread index, opaque to the compiler: a persistent kernel's task loop
// otherwise keeps the addresses that each of its phases derives from it in
// registers over all the other phases (and spills).  For workgroups of 256
// threads; the mask tells the compiler the range, without which it cannot fold
// offsets into LDS addresses.
__device__ __forceinline__ int task_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t & 255;
}

__device__ inline double coherent_load(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void coherent_store(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Publication by value: what a vector holds before its values are published, a
// signalling NaN, which no arithmetic returns.
constexpr unsigned long long SENTINEL = 0x7FF0DEAD00000001ull;
__device__ inline bool is_sentinel(double v) {
  return __builtin_bit_cast(unsigned long long, v) == SENTINEL;
}

// Workgroup barrier for data exchanged through LDS only: waits for this
// wave's LDS operations, not for its global loads and stores in flight (the
// barrier of __syncthreads also waits for those, which puts the latency of
// every write-through store of a published value on the chain).
__device__ inline void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

constexpr long SPIN_LIMIT_DF = 1L << 24;

// Cross-workgroup publication protocol.  Tiles, tile inverses and solve
// vectors are written with agent-coherent (write-through) stores; after every
// thread's stores have completed (s_waitcnt vmcnt(0)) and a barrier, one
// thread stores the ready flag.  Consumers poll flags with agent-coherent
// loads.  Published data is immutable for the rest of the launch, its cache
// lines are never touched before publication by other workgroups (tiles are
// 128-byte aligned: leading dimensions are multiples of 16 doubles, and the
// owner reads its input tile with coherent loads), so plain cached loads of
// published data cannot see stale lines and no cache invalidation is needed.
__device__ inline void wait_stores() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

__device__ inline bool df_wait(const int* f, int epoch, int* err) {
  long spins = 0;
  while (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != epoch) {
    if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
    __builtin_amdgcn_s_sleep(1);
    if (++spins > SPIN_LIMIT_DF) {
      atomicExch(err, 1);
      return false;
    }
  }
  return true;
}

__device__ inline void publish_flag(int* f, int epoch) {
  wait_stores();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(f, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace pdk
