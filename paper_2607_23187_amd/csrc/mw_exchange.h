// Exchange between workgroups of one launch that share an XCD: loads and stores that meet in
// its L2, a counter barrier with a bounded wait, and the placement check at the start.
// Workgroup i of a launch runs on XCD i mod 8; the grid is 8 G and only the workgroups of
// XCD 0 work.  Included by the kernel files only.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "kernels.h"

namespace je {

constexpr int kMwStride = 8;            // XCDs: workgroup i runs on XCD i % 8
constexpr int kMwSpinLimit = 1 << 22;   // polls of one wait before it gives up

__device__ __forceinline__ double ld_ag(const double* p) {
  const unsigned long long v = __hip_atomic_load(
      reinterpret_cast<unsigned long long*>(const_cast<double*>(p)), __ATOMIC_RELAXED,
      __HIP_MEMORY_SCOPE_AGENT);
  return __longlong_as_double((long long)v);
}

// Stores need only reach the L2 that every workgroup of the launch shares (they all run on
// one XCD, checked at the start): workgroup-scope stores are acknowledged there, without
// the write-through of device-scope ones (measured 0.81 against 1.08 us per exchange round
// for 16 workgroups).  Readers use agent-scope loads, which miss their own CU's cache.
__device__ __forceinline__ void st_ag(double* p, double v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p),
                     (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ int ld_ag_i(int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void st_ag_i(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The same for a word: a flag behind stores that have been acknowledged.
__device__ __forceinline__ void st_word(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Arrival of this workgroup at exchange round `round` (1-based) and the wait for all G.
// False when the wait ran out or another workgroup gave up (the abort flag is then set).
__device__ __forceinline__ bool mw_sync(MwCtl* mc, int G, int round) {
  int ok = 1;
  // this wave's stores (its slot and its part of A) have been acknowledged by L2; the
  // compiler fences keep every memory access of the round on its side of the barrier
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(&mc->counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int target = G * round;
    int spins = 0;
    for (;;) {
      // the counter and, behind it, the abort flag
      const unsigned long long v =
          __hip_atomic_load(reinterpret_cast<unsigned long long*>(mc), __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT);
      if ((int)(v & 0xffffffffull) >= target) break;
      if (++spins > kMwSpinLimit || (v >> 32)) {
        st_ag_i(&mc->abort, 1);
        ok = 0;
        break;
      }
    }
  }
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  return __builtin_amdgcn_readfirstlane(ok) != 0;
}

// Start: every workgroup resident and on one XCD, else false with nothing touched (the host
// runs the one-workgroup kernel instead).
__device__ __forceinline__ bool mw_start(MwCtl* mc, int G, int g, int round) {
  const int lane = threadIdx.x;
  if (lane == 0) st_ag_i(&mc->xcc[g], __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 0xf);
  if (!mw_sync(mc, G, round)) {
    if (lane == 0) st_ag_i(&mc->misplaced, 1);
    return false;
  }
  const int x0 = ld_ag_i(&mc->xcc[0]);
  const int xi = lane < G ? ld_ag_i(&mc->xcc[lane]) : x0;
  if (__ballot(xi != x0)) {
    if (g == 0 && lane == 0) st_ag_i(&mc->misplaced, 1);
    return false;
  }
  return true;
}

}  // namespace je
