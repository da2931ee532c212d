// math_probe.hip -- the inner functions of planck_device.hpp evaluated on the
// device, element by element, so that the tests can measure their errors in
// the form that the kernels run.  Not part of libmgrhd.so.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "planck_device.hpp"

namespace mgrhd {

enum Probe : int {
  PROBE_RCP = 0, PROBE_DIV, PROBE_LOG, PROBE_1ME, PROBE_EXP_NEG, PROBE_SQRT, PROBE_STIM,
  PROBE_MEAN, PROBE_MEAN_FIXED, PROBE_COUNT
};

__device__ double probe(int which, double a, double b, double c, double d) {
  switch (which) {
    case PROBE_RCP: return rcp_nr(a);
    case PROBE_DIV: return div_nr(a, b);
    case PROBE_LOG: return log_pos(a);
    case PROBE_1ME: return one_minus_exp(a).em;
    case PROBE_EXP_NEG: return b > 0.0 ? one_minus_exp(a).e : exp_neg(a);
    case PROBE_SQRT: return sqrt_1_4(a);
    case PROBE_STIM: return stim_factor(planck_edge(a));
    case PROBE_MEAN: return mean_ratio_rac(a, b, c, d);
    default: return mean_fixed_rac(a, b);
  }
}

__global__ void k_probe(int which, const double* __restrict__ in, double* __restrict__ out,
                        int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = probe(which, in[i], in[n + i], in[2 * n + i], in[3 * n + i]);
}

}  // namespace mgrhd

// out[n] = function `which` of the four rows of in[4][n] (device pointers)
extern "C" int mgrhd_math_probe(int which, const double* in, double* out, int64_t n,
                                hipStream_t stream) {
  if (which < 0 || which >= mgrhd::PROBE_COUNT || !in || !out || n < 0) return -1;
  if (n == 0) return 0;
  const int64_t blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
  hipLaunchKernelGGL(mgrhd::k_probe, dim3((unsigned)blocks), dim3(256), 0, stream, which, in, out,
                     n);
  return (int)hipGetLastError();
}
