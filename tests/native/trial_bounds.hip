// trial_bounds.hip -- trial_bound (vsh_shower.hpp) at every float that a
// uniform can round to, against the exact distance of the trial.
#include <hip/hip_runtime.h>

#include "vsh_math.hpp"
#include "vsh_shower.hpp"

namespace {

constexpr uint32_t kFirst = 0x25000000u, kLast = 0x3F800000u;  // 2^-53 .. 1: what (2 m + 1) 2^-53 rounds to
constexpr int kMaxCoefs = 32;

struct Coefs {
  double c[kMaxCoefs];
  int n, inverse;  // inverse: the coefficient is c and its reciprocal taken in single precision
};
struct Found {
  unsigned long long above;  // (float, coefficient) pairs whose bound is above the exact distance
  uint32_t worst_bits;       // largest bound over exact distance below 1, as float bits
};

__global__ void __launch_bounds__(256) k_sweep(Coefs k, Found* found) {
  unsigned long long above = 0;
  float worst = 0.0f;
  for (uint64_t b = kFirst + (uint64_t)blockIdx.x * 256 + threadIdx.x; b <= kLast; b += (uint64_t)gridDim.x * 256) {
    const double f = (double)__uint_as_float((uint32_t)b);
    const double next = (double)__uint_as_float((uint32_t)b + 1u);
    // the largest uniform that rounds to f: the one closest to the scale
    const double u = fmin(0.5 * (f + next), 1.0 - 0x1p-53);
    const double dist = -log1p(u - 1.0) / 0.69314718055994530942;  // |log2 u|; u - 1 is exact from 1/2 on
    const double exact = u < 0.5 ? -log2(u) : dist;
    for (int q = 0; q < k.n; ++q) {
      const double ia = k.inverse ? 1.0 / k.c[q] : k.c[q];
      const float ifl = k.inverse ? __builtin_amdgcn_rcpf((float)k.c[q]) : (float)k.c[q];
      const double bound = (double)__uint_as_float(vsh::trial_bound(f, ifl));
      const double ratio = bound / (exact * ia);
      if (ratio > 1.0) ++above;
      else worst = fmaxf(worst, (float)ratio);
    }
  }
  if (above) atomicAdd(&found->above, above);
  atomicMax(&found->worst_bits, __float_as_uint(worst));
}

}  // namespace

extern "C" int trial_bound_sweep(const double* coefs, int n, int inverse, unsigned long long* above, float* worst) {
  if (n < 1 || n > kMaxCoefs) return -1;
  Coefs k{};
  for (int q = 0; q < n; ++q) k.c[q] = coefs[q];
  k.n = n;
  k.inverse = inverse;
  Found* dev = nullptr;
  Found host{};
  if (hipMalloc(&dev, sizeof host) != hipSuccess) return -2;
  hipError_t err = hipMemcpy(dev, &host, sizeof host, hipMemcpyHostToDevice);
  if (err == hipSuccess) {
    hipLaunchKernelGGL(k_sweep, dim3(8192), dim3(256), 0, nullptr, k, dev);
    err = hipGetLastError();
  }
  if (err == hipSuccess) err = hipMemcpy(&host, dev, sizeof host, hipMemcpyDeviceToHost);
  (void)hipFree(dev);
  if (err != hipSuccess) return -3;
  *above = host.above;
  __builtin_memcpy(worst, &host.worst_bits, 4);
  return 0;
}
