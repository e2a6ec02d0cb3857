// Device pieces of the K-SVM recurrence shared by its kernels.
#pragma once

#include "common.hpp"

namespace kdcd {

__device__ __forceinline__ double readlane_d(double v, int l)
{
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)bits, l);
    const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The projected coordinate step of Algorithms 1-2: theta = clip(rho - g/eta, 0, nu) - rho when
// the projected gradient |clip(rho - g, 0, nu) - rho| is non-zero and eta > 0, else 0.
// inv_eta = 1/eta is precomputed (0 when eta <= 0); the selection is branch-free.
__device__ __forceinline__ double dcd_theta(double rho, double g, double inv_eta, double nu)
{
    const double gt = fmin(fmax(rho - g, 0.0), nu) - rho;
    const double th = fmin(fmax(rho - g * inv_eta, 0.0), nu) - rho;
    return (gt != 0.0 && inv_eta > 0.0) ? th : 0.0;
}

}  // namespace kdcd
