// The device forms of the FP64 solver's own elementary routines
// (gks_device.hpp), one launch per call, for tests/test_gpu_device_math.py.
// Host builds of the header compile 1.0 / x and sqrt(x) in their place.
#include <hip/hip_runtime.h>

#include "../paper_2606_17772_amd/csrc/gks_device.hpp"

namespace {
__global__ __launch_bounds__(256) void k_math(int op, const double* __restrict__ x, double* __restrict__ y, int n) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n) return;
  double E, o;
  if (op == 0) y[t] = fdk::m_recip(x[t]);
  else if (op == 1) y[t] = fdk::m_sqrt_normal(x[t]);
  else if (op == 2 || op == 3) {
    fdk::exp_neg(x[t], E, o);
    y[t] = op == 2 ? E : o;
  } else if (op == 4) y[t] = fdk::half_erf_small(x[t]);
  else y[t] = fdk::g_tanh(x[t]);
}
}  // namespace

// x, y: device arrays of n doubles; on the null stream.
extern "C" int device_math(int op, const double* x, double* y, int n) {
  if (op < 0 || op > 5 || n < 1 || !x || !y) return -1;
  hipLaunchKernelGGL(k_math, dim3((n + 255) / 256), dim3(256), 0, nullptr, op, x, y, n);
  return (int)hipGetLastError();
}
