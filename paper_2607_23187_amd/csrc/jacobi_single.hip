// FP64 pivoted Jacobi phase of one matrix on one workgroup.
#include <hip/hip_runtime.h>

#include "jacobi_wg.h"

namespace je {

template <int NT, int RM, bool GAP, bool LDSA, bool MIR, bool SPEC>
__global__ __launch_bounds__(NT) void k_jacobi(JDesc d, long long log_base) {
  jacobi_run<NT, RM, GAP, LDSA, MIR, false, SPEC>(d, log_base);
}

static int g_max_lds = -1;

static int max_lds() {
  if (g_max_lds < 0) {
    int dev = 0, v = 65536;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess)
      g_max_lds = v;
    else
      g_max_lds = 65536;
  }
  return g_max_lds;
}

bool jacobi_fits_lds(int n) {
  return n <= 128 && jacobi_lds_bytes(n, true) + 8192 <= (size_t)max_lds();
}

template <int NT, int RM, bool GAP, bool LDSA, bool MIR>
static hipError_t launch_one(const JDesc& d, long long log_base, hipStream_t s) {
  // thread tid owns rows tid + i NT, i < RM: every row of the matrix needs an owner
  if ((long long)NT * RM < d.n) return hipErrorInvalidValue;
  size_t sh = jacobi_lds_bytes(d.n, LDSA);
  auto fn = spec_depth<RM, false>() > 0 && jacobi_speculates(d.pivot, d.stop)
                ? k_jacobi<NT, RM, GAP, LDSA, MIR, (spec_depth<RM, false>() > 0)>
                : k_jacobi<NT, RM, GAP, LDSA, MIR, false>;
  if (sh > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)fn,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(fn, dim3(1), dim3(NT), sh, s, d, log_base);
  return hipGetLastError();
}

// Threads per workgroup for the HBM-resident kernel: 512 (two waves per SIMD, 256 VGPRs
// per lane); rows per thread RM = ceil(n / NT).
template <bool GAP, bool MIR>
static hipError_t launch_global(const JDesc& d, long long log_base, hipStream_t s) {
  const int n = d.n;
  if (n <= 256) return launch_one<256, 1, GAP, false, MIR>(d, log_base, s);
  if (n <= 512) return launch_one<512, 1, GAP, false, MIR>(d, log_base, s);
  if (n <= 1024) return launch_one<512, 2, GAP, false, MIR>(d, log_base, s);
  if (n <= 2048) return launch_one<512, 4, GAP, false, MIR>(d, log_base, s);
  if (n <= 4096) return launch_one<512, 8, GAP, false, MIR>(d, log_base, s);
  return launch_one<1024, 8, GAP, false, MIR>(d, log_base, s);
}

// HBM-resident matrices: mirror mode (rows and columns p, q stored, every load a contiguous
// row segment) or timestamp mode (rows only, the newer copy of each entry chosen by per-row
// write timestamps).  Both give the same arithmetic and the same pivot sequence.
template <bool GAP>
static hipError_t launch_jacobi_t(const JDesc& d, long long log_base, bool lds, bool mirror,
                                  hipStream_t s) {
  const int n = d.n;
  if (lds) {
    if (n <= 64) return launch_one<64, 1, GAP, true, true>(d, log_base, s);
    return launch_one<64, 2, GAP, true, true>(d, log_base, s);
  }
  if (mirror) return launch_global<GAP, true>(d, log_base, s);
  return launch_global<GAP, false>(d, log_base, s);
}

hipError_t launch_jacobi(const JDesc& d, long long log_base, bool lds_mode, bool mirror,
                         hipStream_t s) {
  if (d.pivot == 1) return launch_jacobi_t<true>(d, log_base, lds_mode, mirror, s);
  return launch_jacobi_t<false>(d, log_base, lds_mode, mirror, s);
}

}  // namespace je
