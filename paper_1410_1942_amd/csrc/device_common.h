// What both device files use: typed global-memory views, the refined
// reciprocal and the face coefficient, and a slot's direction buffers.
#ifndef PCG_DEVICE_COMMON_H
#define PCG_DEVICE_COMMON_H

#include <hip/hip_runtime.h>
#include <math.h>

#include "pcg_types.h"

namespace pcgmi {

// Global-address-space views: pointers read from the slot table are
// generic; casting them lets the compiler emit global (not flat) accesses.
#define GLB __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ GLB T *gp(T *p) { return (GLB T *)p; }
template <typename T>
__device__ __forceinline__ const GLB T *gp(const T *p) { return (const GLB T *)p; }

__device__ __forceinline__ void *dir_buf(const Slot &S, int b)
{
    return b == 0 ? S.dir0 : (b == 1 ? S.dir1 : S.dir2);
}

// Reciprocal of a positive finite value: hardware estimate refined by two
// Newton-Raphson steps (quadratic convergence from the ~2^-23 estimate).
__device__ __forceinline__ double recip(double d)
{
    double y = __builtin_amdgcn_rcp(d);
    double e = fma(-d, y, 1.0);
    y = fma(y, e, y);
    e = fma(-d, y, 1.0);
    return fma(y, e, y);
}
__device__ __forceinline__ float recip(float d) { return __builtin_amdgcn_rcpf(d); }

// Face coefficient from the sum of the two densities on either side:
// beta = 1/((rho_c + rho_n)/2) = 2/(rho_c + rho_n).  A hull cell holds +inf,
// so the sum is +inf and beta = 0.  Walls use rho_n = 0 for Dirichlet
// (beta = 2/rho_c: the mirrored ghost -p_c) and +inf for Neumann (beta = 0).
template <typename T>
__device__ __forceinline__ T fb(T den)
{
    const T inf = (T)INFINITY;
    return den < inf ? T(2) * recip(den) : T(0);
}

// A power of two near 1/norm, so that scaling by it is exact.
__device__ __forceinline__ double pow2_scale(double norm)
{
    if (!(norm > 0.0) || !isfinite(norm)) return 1.0;
    return ldexp(1.0, -ilogb(norm));
}

}  // namespace pcgmi

#endif
