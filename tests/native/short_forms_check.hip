// Every float of their ranges through the short square root and reciprocal,
// against the float64 functions rounded once (a float64 root or quotient rounded
// to float32 is the correctly rounded one: 53 >= 2 * 24 + 2 bits); every float
// through the exact_ forms; and every positive float as a bound through
// radius_limit.  Prints one line per check, "ok" last when no float differs.
#include <stdio.h>

#include "../../paper_2403_09990_amd/csrc/purse_traj.hpp"

using namespace purse;

constexpr int kChecks = 5;
struct Count {
  unsigned long long tried[kChecks], differ[kChecks];
};

__device__ bool same(float a, float b) {
  return __float_as_uint(a) == __float_as_uint(b) || (a != a && b != b);
}

__global__ void k_check(Count *out) {
  unsigned long long tried[kChecks] = {}, differ[kChecks] = {};
  const unsigned long long step = (unsigned long long)gridDim.x * blockDim.x;
  for (unsigned long long u = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; u < (1ull << 32); u += step) {
    const float x = __uint_as_float((unsigned)u);
    const float root = (float)sqrt((double)x), rcp = (float)(1.0 / (double)x);
    if (x >= kShortMin && x <= kShortMax) {
      ++tried[0];
      differ[0] += !same(short_sqrt(x), root);
    }
    if (fabsf(x) >= kShortMin && fabsf(x) <= kShortMax) {
      ++tried[1];
      differ[1] += !same(short_rcp(x), rcp);
    }
    ++tried[2];
    differ[2] += !same(exact_sqrt(x), sqrtf(x));
    ++tried[3];
    differ[3] += !same(exact_rcp(x), 1.f / x);
    if (x >= 0.f) {
      // the largest squared radius whose root is at most x
      const float t = radius_limit(x);
      const bool in = sqrtf(t) <= x, last = !(t < FLT_MAX) || sqrtf(__uint_as_float(__float_as_uint(t) + 1u)) > x;
      ++tried[4];
      differ[4] += !(in && last);
    }
  }
  for (int k = 0; k < kChecks; ++k) {
    atomicAdd(&out->tried[k], tried[k]);
    atomicAdd(&out->differ[k], differ[k]);
  }
}

int main() {
  const char *names[kChecks] = {"short_sqrt", "short_rcp", "exact_sqrt", "exact_rcp", "radius_limit"};
  Count *dev = nullptr, host = {};
  if (hipMalloc(&dev, sizeof host) != hipSuccess ||
      hipMemcpy(dev, &host, sizeof host, hipMemcpyHostToDevice) != hipSuccess)
    return 1;
  hipLaunchKernelGGL(k_check, dim3(4096), dim3(256), 0, 0, dev);
  if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(&host, dev, sizeof host, hipMemcpyDeviceToHost) != hipSuccess)
    return 1;
  (void)hipFree(dev);
  unsigned long long bad = 0;
  for (int k = 0; k < kChecks; ++k) {
    printf("%-12s %llu floats, %llu differ\n", names[k], host.tried[k], host.differ[k]);
    bad += host.differ[k] + (host.tried[k] == 0);
  }
  if (bad == 0) printf("ok\n");
  return bad ? 2 : 0;
}
