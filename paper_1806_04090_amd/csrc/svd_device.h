// Device helpers shared by the encoders that work in double precision on the Gram matrix (svd_direct.hip, svd_thin.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <type_traits>

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

// ------------------------------------------------------------------------------------------------
// wave helpers (64 lanes, no LDS)
// ------------------------------------------------------------------------------------------------
template <int CTRL>
__device__ inline double dpp(double x)
{
    const unsigned a = (unsigned)__builtin_amdgcn_mov_dpp((int)lo32(x), CTRL, 0xf, 0xf, true);
    const unsigned b = (unsigned)__builtin_amdgcn_mov_dpp((int)hi32(x), CTRL, 0xf, 0xf, true);
    return mk64(a, b);
}
// what lane L of the lane's row of 16 holds (both halves in one instruction: the only control that 64-bit moves have)
template <int L>
__device__ inline double row_lane(double x)
{
    return __longlong_as_double((long long)__builtin_amdgcn_mov_dpp(__double_as_longlong(x), 0x150 + L, 0xf, 0xf, true));
}
// ... in the fours of lanes of BANKS, and `other` in the rest
template <int L, int BANKS>
__device__ inline double row_lane(double other, double x)
{
    return __longlong_as_double((long long)__builtin_amdgcn_update_dpp(__double_as_longlong(other), __double_as_longlong(x), 0x150 + L, 0xf, BANKS, false));
}
// The value is worked out where this stands and not where it is used first (behind a wait, as a rule).
__device__ inline void here(double& x) { asm volatile("" : "+v"(x)); }
// acc +- (what lane L of the lane's row of 16 holds of b) * x in one instruction, rounded once.  b has to come out of `broadcasts`: between
// the instruction that writes it and the first of these are two wait states, and the compiler does not know what is inside (the built
// code is looked over in a test).
__device__ inline void wait_for_broadcasts() { asm volatile("s_nop 1"); }
template <typename... D>
__device__ inline void broadcasts(D&... b)
{
    (here(b), ...);
    wait_for_broadcasts();
    (here(b), ...);
}
template <int L>
__device__ inline void add_lane_product(double& acc, double b, double x)
{
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(b), "v"(x), "n"(L));
}
template <int L>
__device__ inline void sub_lane_product(double& acc, double b, double x)
{
    asm("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(b), "v"(x), "n"(L));
}
// f(integral_constant 0) .. f(integral_constant 15)
template <int L = 0, typename F>
__device__ inline void for_lanes(F&& f)
{
    if constexpr (L < 16) {
        f(std::integral_constant<int, L>());
        for_lanes<L + 1>(f);
    }
}
constexpr int DPP_SHL1 = 0x101, DPP_SHL2 = 0x102, DPP_SHL4 = 0x104, DPP_SHL8 = 0x108;    // lane l: what lane l + n of its row has, or 0
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140, DPP_ROR8 = 0x128;

// lanes 0..31 of the result: a of the lane plus a of lane + 32; lanes 32..63: b of both
__device__ inline double fold32(double a, double b)
{
    const auto l = __builtin_amdgcn_permlane32_swap(lo32(a), lo32(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi32(a), hi32(b), false, false);
    return mk64(l[0], h[0]) + mk64(l[1], h[1]);
}
// the same between neighbouring rows of 16 lanes (even rows: a, odd rows: b)
__device__ inline double fold16(double a, double b)
{
    const auto l = __builtin_amdgcn_permlane16_swap(lo32(a), lo32(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi32(a), hi32(b), false, false);
    return mk64(l[0], h[0]) + mk64(l[1], h[1]);
}
__device__ inline double sum8(double x)      // over the 8 lanes of a group, in every lane
{
    x += dpp<DPP_XOR1>(x);
    x += dpp<DPP_XOR2>(x);
    x += dpp<DPP_HALF_MIRROR>(x);
    return x;
}
// sum over the 64 lanes, the same bits in every lane
__device__ inline double wave_sum(double x)
{
    x = sum8(x);
    x += dpp<DPP_MIRROR>(x);
    x = fold16(x, x);
    return fold32(x, x);
}

__device__ inline double lane_value(double x, int lane)
{
    return mk64((unsigned)__builtin_amdgcn_readlane((int)lo32(x), lane), (unsigned)__builtin_amdgcn_readlane((int)hi32(x), lane));
}

// Step k: x = column k of the current matrix, v the Householder vector that maps x[k + 1 ..] to a multiple of the first
// unit vector, p = A v, w = tau p - (tau^2 / 2)(v^T p) v, A <- A - v w^T - w v^T.
// beta, the entry that remains, and v_{k+1} = alpha - beta; tau = 2 / v^T v.  (A column of zeros: the floor under the
// root makes v a multiple of the first unit vector and the step a change of sign.  The trace is about 1.)
__device__ inline void householder(double alpha, double sig2, double& beta, double& v0)
{
    beta = -copysign(root(fma(alpha, alpha, fmax(sig2, 1e-150))), alpha);
    v0 = alpha - beta;
}
__device__ inline double householder_tau(double sig2, double v0) { return 2.0 * reciprocal(fma(v0, v0, sig2)); }

// The search for eigenvalues of T (matrices scaled to a trace under 1), in cells of equal relative width.
constexpr double OD2_MIN = 7.7e-34;          // 2^-110: keeps the Sturm recurrence going where T splits
constexpr double FLOOR_REL = 1.4551915e-11;  // 2^-36: four times the squared fp32 floor of the encoder (ZERO_REL)
constexpr int LAM_BITS = 27;                 // the search ends at this relative precision of lambda
constexpr u64 LAM_MIN_BITS = 0x3CD0000000000000ull;   // 2^-50: anything below is zero (lambda_1 >= 2^-12 in this scale)
constexpr u64 LAM_MAX_BITS = 0x3FF0000000000000ull;   // 1.0: the trace is below it
constexpr int LAM_STEP_BITS = 52 - LAM_BITS;

__device__ inline double bits_double(u64 b) { return __longlong_as_double((long long)b); }

__device__ inline double cell_start(u64 cell) { return bits_double(LAM_MIN_BITS + (cell << LAM_STEP_BITS)); }

// When the vectors of kept atoms are orthogonal.  Two vectors with residuals res of eigenvalues a distance `gap` apart have
// a cosine of up to 2 res / gap, and their images on the other side one of about res / (sigma_i sigma_j) more, so a residual
// that is small against the largest eigenvalue says nothing about atoms far below it.  What is asked for:
//   - a residual, together with the rounding of the factorisation (every entry of T to an ulp or two: `weight`, the sum of
//     |T_ij| z_i^2, times 2^-52), under 2e-5 of both distances;
//   - a Rayleigh quotient that has stayed with its own eigenvalue: in a cluster two vectors can end at the same one;
//   - eigenvalues further apart than what the search resolves (`cells` of the smaller).
// Neighbours are those among the kept atoms: directions that the message does not hold may mix.  One dominant singular
// value over a tail of equal ones, 1e-3 to 1e-5 of it, rounded to fp32, 6 x 900 to 300 x 400: with a bound on the residual alone
// cosines up to 1; with these up to 8e-6 (the others are left over).  Noise spectra, neighbours of their bulk included: none left over.
struct KeptApart {
    double lam, gap, product;        // distance to the nearest neighbour; sigma_i sigma_j squared for the one before
    bool possible;
    // up, down: eigenvalues of the kept atoms before and after this one, negative if there is none
    __device__ inline KeptApart(double own, double up, double down, double cells) : lam(own)
    {
        gap = fmin(up >= 0.0 ? up - own : 1e300, down >= 0.0 ? own - down : 1e300);
        product = up >= 0.0 ? up * own : 1e300;
        possible = (up < 0.0 || up - own > cells * own) && (down < 0.0 || own - down > cells * down);
    }
    __device__ inline bool vector(double residual, double weight, double rayleigh) const
    {
        const double e = fma(weight, 2.220446049250313e-16, residual);
        return possible && e <= 2e-5 * gap && e * e <= 4e-10 * product && fabs(rayleigh - lam) <= 0.25 * gap;
    }
};

}  // namespace atomo
