// Sums over the lanes of a wave, and scalars handed between blocks past the L2.
#pragma once

// Values to have been requested here (a uniform branch on one of them would otherwise wait
// for its own round trip to memory before the others are asked for).
#define LOADED(a, b) asm volatile("" ::"s"(a), "s"(b))

#include <hip/hip_runtime.h>
#include <stdint.h>

// Sum over the wave's 64 lanes in a fixed order (row shifts, then the row broadcasts of
// the data-parallel primitives: no LDS round trips); the total is in lane 63.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xF, false);
  return v + __builtin_bit_cast(double, ((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
}
__device__ __forceinline__ double wave_sum63(double v) {
  v = dpp_add<0x111, 0xF>(v);  // row_shr:1
  v = dpp_add<0x112, 0xF>(v);  // row_shr:2
  v = dpp_add<0x114, 0xF>(v);  // row_shr:4
  v = dpp_add<0x118, 0xF>(v);  // row_shr:8
  v = dpp_add<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Stores and loads at agent scope: written through to, and read from, the memory the eight
// L2 caches share, so no block has to write its cache back.  arrive() waits for the wave's
// stores and counts it (one lane); every scalar of the blocks that arrived before is visible.
__device__ __forceinline__ void put_agent(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get_agent(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned arrive(unsigned* counter) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
