// Test library: the scalar functions of the stages on the GPU, beside the
// library functions in whose place they stand.
#include <hip/hip_runtime.h>

#include "dimp_device.hpp"

namespace {

enum { FRCP, QUOT, FSQRT, TIMES_INVERSE, EXP_CURVE, LIB_EXP };

__global__ void k_scalar(int fn, int n, const double* a, const double* b, double* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = a[i], y = b[i];
  double r = 0.0;
  if (fn == FRCP) r = dimp::frcp(y);
  if (fn == QUOT) r = dimp::quot(x, y);
  if (fn == FSQRT) r = dimp::fsqrt(y);
  if (fn == TIMES_INVERSE) {  // the inverse as the host packs it
    const double i0 = 1.0 / y;
    r = dimp::times_inverse(x, i0, fma(-i0, y, 1.0) / y);
  }
  if (fn == EXP_CURVE) r = dimp::exp_curve(x);
  if (fn == LIB_EXP) r = exp(x);
  out[i] = r;
}

}  // namespace

extern "C" int scalar_run(int fn, int n, const double* a, const double* b, double* out) {
  hipLaunchKernelGGL(k_scalar, dim3((n + 255) / 256), dim3(256), 0, nullptr, fn, n, a, b, out);
  return hipDeviceSynchronize() != hipSuccess;
}
