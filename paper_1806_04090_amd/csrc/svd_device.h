// Device helpers shared by the encoders that work in double precision on the Gram matrix (svd_direct.hip, svd_thin.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace atomo {

typedef unsigned long long u64;
typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

// A pointer out of a descriptor as one into global memory: the compiler cannot know that, and a load through a generic
// pointer waits for the LDS as well.
template <typename T>
using Global = T __attribute__((address_space(1)))*;
template <typename T>
__device__ inline Global<T> global(T* p) { return (Global<T>)p; }

__device__ inline unsigned lo32(double x) { return (unsigned)__double_as_longlong(x); }
__device__ inline unsigned hi32(double x) { return (unsigned)(__double_as_longlong(x) >> 32); }
__device__ inline double mk64(unsigned lo, unsigned hi) { return __longlong_as_double((long long)(((u64)hi << 32) | lo)); }

// Square root and reciprocal of a positive normal number, to the last bits: the hardware's estimates, then Goldschmidt's and
// Newton's iterations (no scaling, no special cases: half the latency of sqrt() and of a division in a serial chain).
__device__ inline double root(double x)
{
    const double r = __builtin_amdgcn_rsq(x);
    double g = x * r, h = 0.5 * r;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double e = fma(-h, g, 0.5);
        g = fma(g, e, g);
        h = fma(h, e, h);
    }
    return fma(fma(-g, g, x), h, g);
}
__device__ inline double reciprocal(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

}  // namespace atomo
