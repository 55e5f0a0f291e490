// FP64 pivoted Jacobi phase of a batch: persistent workgroups over a queue of matrices.
#include <hip/hip_runtime.h>

#include "jacobi_wg.h"

namespace je {

// Persistent form for a batch: each workgroup takes the next matrix from a device counter
// (the host orders idx largest first) and runs the same pivoted Jacobi on it, until the
// list is exhausted.  Workgroups never wait for each other.
template <int NT, int RM, bool GAP, bool LDSA, bool MIR, bool SPEC>
__global__ __launch_bounds__(NT) void k_jacobi_queue(BMat* __restrict__ mats,
                                                     const int* __restrict__ idx, int count,
                                                     int* counter) {
  __shared__ int s_next;
  for (;;) {
    __syncthreads();  // the previous matrix is finished with LDS
    if (threadIdx.x == 0) s_next = atomicAdd(counter, 1);
    __syncthreads();
    const int t = s_next;
    if (t >= count) return;
    const BMat& b = mats[idx[t]];
    jacobi_run<NT, RM, GAP, LDSA, MIR, true, SPEC>(b.jd, b.log_base);
  }
}

template <int NT, int RM, bool GAP, bool LDSA>
static hipError_t launch_queue_one(BMat* m, const int* idx, int count, int nmax, bool spec,
                                   bool mirror, int* counter, int grid, hipStream_t s) {
  if ((long long)NT * RM < nmax) return hipErrorInvalidValue;
  size_t sh = jacobi_lds_bytes(nmax, LDSA);
  constexpr bool kSpec = spec_depth<RM, true>() > 0;
  auto fn = (LDSA || mirror) ? (spec ? k_jacobi_queue<NT, RM, GAP, LDSA, true, kSpec>
                                     : k_jacobi_queue<NT, RM, GAP, LDSA, true, false>)
                             : (spec ? k_jacobi_queue<NT, RM, GAP, LDSA, LDSA, kSpec>
                                     : k_jacobi_queue<NT, RM, GAP, LDSA, LDSA, false>);
  // under graph capture the attribute was set by a preparing call (grid 0) beforehand
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) != hipSuccess) return hipGetLastError();
  if (sh > 65536 && cs == hipStreamCaptureStatusNone) {
    hipError_t e = hipFuncSetAttribute((const void*)fn,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
  }
  if (grid <= 0) return hipSuccess;  // attributes only (before a graph capture)
  hipLaunchKernelGGL(fn, dim3(grid), dim3(NT), sh, s, m, idx, count, counter);
  return hipGetLastError();
}

// Workgroup shapes of the batched Jacobi: LDS-resident matrices (n <= 128) with one or two
// waves, HBM-resident ones with 128, 256 or 512 threads (128 and 256 up to n = 512; 1024
// threads above n = 4096); rows per thread = ceil(nmax / threads).
template <bool GAP>
static hipError_t launch_queue_t(BMat* m, const int* idx, int count, int nmax, bool lds,
                                 bool spec, bool mirror, int threads, int* counter, int grid,
                                 hipStream_t s) {
  if (lds) {
    if (threads == 128 && nmax <= 128)
      return launch_queue_one<128, 1, GAP, true>(m, idx, count, nmax, spec, mirror, counter, grid, s);
    if (nmax <= 64)
      return launch_queue_one<64, 1, GAP, true>(m, idx, count, nmax, spec, mirror, counter, grid, s);
    return launch_queue_one<64, 2, GAP, true>(m, idx, count, nmax, spec, mirror, counter, grid, s);
  }
  if (threads == 256) {
    if (nmax <= 256)
      return launch_queue_one<256, 1, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
    if (nmax <= 512)
      return launch_queue_one<256, 2, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
  }
  if (threads == 128) {
    if (nmax <= 128)
      return launch_queue_one<128, 1, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
    if (nmax <= 256)
      return launch_queue_one<128, 2, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
    if (nmax <= 512)
      return launch_queue_one<128, 4, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
  }
  if (nmax <= 512)
    return launch_queue_one<512, 1, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
  if (nmax <= 1024)
    return launch_queue_one<512, 2, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
  if (nmax <= 2048)
    return launch_queue_one<512, 4, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
  if (nmax <= 4096)
    return launch_queue_one<512, 8, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
  return launch_queue_one<1024, 8, GAP, false>(m, idx, count, nmax, spec, mirror, counter, grid, s);
}

hipError_t launch_jacobi_queue(BMat* m, const int* idx, int count, int nmax, int pivot,
                               int stop, bool lds_mode, bool mirror, int threads, int* counter, int grid,
                               hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const bool spec = jacobi_speculates(pivot, stop);
  if (pivot == 1)
    return launch_queue_t<true>(m, idx, count, nmax, lds_mode, spec, mirror, threads, counter, grid, s);
  return launch_queue_t<false>(m, idx, count, nmax, lds_mode, spec, mirror, threads, counter, grid, s);
}

}  // namespace je
