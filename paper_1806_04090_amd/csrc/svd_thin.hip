// Spectral-ATOMO encode of thin matrices: at most 32 vectors on the shorter side, any number of positions on the longer one
// (a convolution gradient [x, y, k, k] in the reshape [x y / 2, 2 k k] of Section 6 has 18 columns).
//
// Three launches and two passes over the data:
//     thin_gram  : partial r x r Gram matrices of runs of positions, in double precision on the matrix cores
//     thin_solve : one workgroup per matrix sums them, takes the singular values of the sum (tridiagonal form and Sturm counts,
//                  or, where that is not accepted, two-sided Jacobi, all in LDS), runs Algorithm 1, draws the mask and
//                  writes the message but for the long vectors
//     thin_long  : the long vectors of the kept atoms, A^T u / sigma
// Products of two floats are exact in double precision: lambda has an absolute error of about 1e-15 lambda_1.  The vectors of
// the direct solution are orthogonal as KeptApart asks, Jacobi's to rounding whatever the spectrum looks like.
#include <algorithm>
#include <vector>

#include "svd_device.h"
#include "svd_thin.h"

namespace atomo {
namespace thin {

using svd::Work;

namespace {

constexpr int GRAM_WAVES = 8;
constexpr int GRAM_CHUNK = 128 * GRAM_WAVES;   // positions per workgroup: eight rounds of 16 per wave
constexpr int MAX_CHUNKS = 128;
constexpr int AHEAD = 3;                       // rounds in flight (80 registers: three workgroups per compute unit, two with 4: 20.5 us)
constexpr int PART = 3 * 256;                  // doubles of a partial Gram matrix

// Bound: the matrix cores, with a 16 x 16 x 4 product per four positions up to 16 vectors, three from there on; vectors 16 .. 19
// (the 18 columns of a 3 x 3 convolution) take two of 4 x 4 x 4 in four blocks, an eighth of the time of the two they replace.
// 11.16 M elements of 18 columns: 19 us (27 with three large products; 14 without any).
__global__ __launch_bounds__(64 * GRAM_WAVES) void thin_gram(const ThinMat* mats, const Work* work)
{
    __shared__ double red[GRAM_WAVES / 2][PART];
    const Work wk = work[blockIdx.x];
    const ThinMat& m = mats[wk.mat];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, q = lane >> 4;
    const int r = m.r, p_end = min(m.M, (wk.a + 1) * m.chunk);
    const bool two = r > 16, narrow = two && r <= 20;
    // entry (vector i, position p) at i * by_vec + p * by_pos; a lane holds vectors l16 and 16 + l16 (clamped: zeroed below)
    const long long by_vec = m.tall ? 1 : m.ldg, by_pos = m.tall ? m.ldg : 1;
    const Global<const float> g0 = global(m.G) + (long long)min(l16, r - 1) * by_vec;
    const int second = 16 + (narrow ? l16 & 3 : l16);
    const Global<const float> g1 = global(m.G) + (long long)min(second, r - 1) * by_vec;
    const float m0 = l16 < r ? 1.0f : 0.0f, m1 = second < r ? 1.0f : 0.0f;
    double cross = 0.0, corner = 0.0;                            // narrow: entries (4 (l16 / 4) + q, second) and (16 + q, second)
    doublex4 acc[3] = {doublex4{0, 0, 0, 0}, doublex4{0, 0, 0, 0}, doublex4{0, 0, 0, 0}};
    // the four positions p0 + 4 q + s of a round, one per instruction; those of the next rounds are on their way meanwhile
    struct Round { float a[4], b[4]; };
    auto fetch = [&](int p0, Round& x) {
        const int p = p0 + 4 * q;
        const Global<const float> h0 = g0 + p * by_pos, h1 = g1 + p * by_pos;
        if (p0 + 16 <= p_end) {
#pragma unroll
            for (int s = 0; s < 4; ++s) x.a[s] = h0[s * by_pos];
            if (two) {
#pragma unroll
                for (int s = 0; s < 4; ++s) x.b[s] = h1[s * by_pos];
            }
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const long long at = min(p + s, m.M - 1) * by_pos;
                x.a[s] = p + s < p_end ? g0[at] : 0.0f;
                x.b[s] = two && p + s < p_end ? g1[at] : 0.0f;
            }
        }
    };
    auto add = [&](const Round& x) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double u = m0 != 0.0f ? (double)x.a[s] : 0.0;
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(u, u, acc[0], 0, 0, 0);
            if (two) {
                const double v = m1 != 0.0f ? (double)x.b[s] : 0.0;
                if (narrow) {
                    // block b: rows 4 b .. 4 b + 3 (lane l16 = 4 b + row, position q) by columns 16 .. 19
                    cross = __builtin_amdgcn_mfma_f64_4x4x4f64(u, v, cross, 0, 0, 0);
                    corner = __builtin_amdgcn_mfma_f64_4x4x4f64(v, v, corner, 0, 0, 0);
                } else {
                    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(u, v, acc[1], 0, 0, 0);
                    acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, v, acc[2], 0, 0, 0);
                }
            }
        }
    };
    constexpr int STEP = 16 * GRAM_WAVES;
    Round x[AHEAD];
    int p0 = wk.a * m.chunk + 16 * wave;
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
        if (p0 + u * STEP < p_end) fetch(p0 + u * STEP, x[u]);
    for (; p0 < p_end; p0 += AHEAD * STEP) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (p0 + u * STEP >= p_end) break;
            add(x[u]);
            if (p0 + (u + AHEAD) * STEP < p_end) fetch(p0 + (u + AHEAD) * STEP, x[u]);
        }
    }
    // the waves' sums in a fixed order: the upper half of them hands its own over, then all add up
    const int tiles = two ? 3 : 1;
    auto give = [&](double* to, bool add) {
        auto put = [&](int e, double x) { to[e] = add ? to[e] + x : x; };
#pragma unroll
        for (int v = 0; v < 4; ++v) put((4 * v + q) * 16 + l16, acc[0][v]);
        if (narrow) {
            put(256 + (l16 & 3) * 16 + 4 * (l16 >> 2) + q, cross);
            if (l16 < 4) put(512 + l16 * 16 + q, corner);
        } else if (two) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                put(256 + l16 * 16 + 4 * v + q, acc[1][v]);
                put(512 + (4 * v + q) * 16 + l16, acc[2][v]);
            }
        }
    };
    if (wave >= GRAM_WAVES / 2) give(red[wave - GRAM_WAVES / 2], false);
    __syncthreads();
    if (wave < GRAM_WAVES / 2) give(red[wave], true);
    __syncthreads();
    const Global<double> out = global(m.part) + (size_t)wk.a * PART;
    for (int f = tid; f < (narrow ? 384 : 256 * tiles); f += 64 * GRAM_WAVES) {
        const int e = narrow && f >= 320 ? f + 192 : f;          // (narrow: four vectors of the second and of the third tile)
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < GRAM_WAVES / 2; ++w) sum += red[w][e];
        out[e] = sum;
    }
}

// ------------------------------------------------------------------------------------------------
constexpr int ST = 512;                        // threads of a workgroup of thin_solve
constexpr int LD = THIN_R + 1;
constexpr int MAX_SWEEPS = 15;

// 1 / sqrt(x) of a positive normal number: the hardware's estimate (23 bits) and one step of third order, two dependent
// operations shorter than two of Newton's.
__device__ inline double inverse_root(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double h = fma(-x * y, y, 1.0);                        // x y^2 = 1 - h
    return fma(y * h, fma(0.375, h, 0.5), y);
}

// Jacobi rotation of the pair with diagonal entries a, b and off-diagonal g: columns (x, y) become (c x - s y, s x + c y),
// rows likewise.  With h = (b - a) / 2 the angle has cos 2 phi = |h| / sqrt(h^2 + g^2) and s has the sign of h g; the
// identity for g = 0.
__device__ inline void rotation(double a, double b, double g, double& c, double& s)
{
    const double h = 0.5 * (b - a), hh = fma(h, h, g * g);
    const bool none = !(hh > 1e-300);
    const double inv = inverse_root(none ? 1.0 : hh);
    const double cc = none ? 1.0 : fma(0.5 * fabs(h), inv, 0.5), ic = inverse_root(cc);
    c = cc * ic;
    s = none ? 0.0 : copysign(0.5, h) * g * inv * ic;
}

// Householder reduction of the n x n matrix C (LDS, both triangles, zeros from n on), n <= 2 U, by one wave: diagonal d, off-diagonal
// e; the vectors of the steps go to the rows of H.  Lane l belongs to row 2 (l mod 16) + (l / 16 mod 2) and holds its columns 2 u + l / 32, u < U,
// in registers.  The column below its first entry and w are operands that are broadcast inside the products: of a vector, every row of
// 16 lanes gets the entries of its columns, which some row of lanes has in this order.  Column k + 1 (the row of that number) goes around
// through LDS, beside the products.  The product is taken with the column without its first entry, under way before the reflector is known
// (A v = A y + v0 A e_{k+1}), and the update by a step stands beside the sums of the next.
// Bound: a chain of about 180 instructions.  18 columns: 1230 cycles per step; 1340 with all sixteen columns per lane, through LDS or not.
struct TriScratch { double column[THIN_R]; };
__device__ inline int tri_lane(int row) { return (row & 1) << 4 | row >> 1; }
template <int U>
__device__ inline void tridiagonal(const double* C, double* H, TriScratch& lds, double* d, double* e, double* tau, int n)
{
    const int lane = threadIdx.x & 63, h = lane >> 5, i = 2 * (lane & 15) + (lane >> 4 & 1);
    auto half_sum = [](double y) {                               // over the 32 lanes of a half, the same bits in each
        y = sum8(y);
        y += dpp<DPP_MIRROR>(y);
        return fold16(y, y);
    };
    auto columns = [](auto&& f) { for_lanes([&](auto u) { if constexpr (decltype(u)::value < U) f(u); }); };
    double a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = C[i * LD + 2 * u + h];
    static_assert(U % 2 == 0, "written in pairs");
    auto put_row = [&](int row) {                                // (for lane l of either half: the entry of its own row)
        if (i == row) {
#pragma unroll
            for (int u = 0; u < U; u += 2) *(doublex2*)&lds.column[16 * h + u] = doublex2{a[u], a[u + 1]};
        }
    };
    // of a vector that both halves of the lanes have: the entry of column 2 j + h in lane j of the row of lanes
    auto spread = [&](double y) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo32(y), lo32(y), false, false);
        const auto g = __builtin_amdgcn_permlane16_swap(hi32(y), hi32(y), false, false);
        return mk64(h ? l[1] : l[0], h ? g[1] : g[0]);
    };
    if (h == 0) lds.column[lane] = 0.0;                          // (what no column is written to)
    double x = C[i * LD];                                        // column k of the current matrix, in both halves
    double v = 0.0, w = 0.0, yj = 0.0, wj = 0.0;                 // the last step's, which the matrix has still to be updated with
    auto update = [&] {
        broadcasts(yj, wj);
        columns([&](auto u) { sub_lane_product<decltype(u)::value>(a[u], yj, w); });
        columns([&](auto u) { sub_lane_product<decltype(u)::value>(a[u], wj, v); });
    };
    for (int k = 0; k + 2 < n; ++k) {
        const double y = i > k + 1 ? x : 0.0;
        const double alpha = lane_value(x, tri_lane(k + 1)), diagonal = lane_value(x, tri_lane(k));
        const double sig2 = half_sum(y * y);
        // (column k + 1, for which y is not v, is not used any more)
        update();
        put_row(k + 1);
        lanes_in_order();
        const double c = lds.column[lane & 31];
        yj = spread(y);
        broadcasts(yj);
        double even = 0.0, odd = 0.0;
        columns([&](auto u) {
            constexpr int J = decltype(u)::value;
            add_lane_product<J>(J & 1 ? odd : even, yj, a[J]);
        });
        double beta, v0;
        householder(alpha, sig2, beta, v0);
        const double t = householder_tau(sig2, v0);
        v = i == k + 1 ? v0 : y;
        const double part = even + odd;
        const double p = i > k ? t * fma(v0, c, fold32(part, part)) : 0.0;
        w = fma(-0.5 * t * half_sum(p * v), v, p);
        wj = spread(w);
        x = fma(-w, v0, fma(-v, lane_value(w, tri_lane(k + 1)), c));
        if (h == 0) H[k * LD + i] = v;
        if (lane == 0) {
            d[k] = diagonal;
            e[k] = beta;
            tau[k] = t;
        }
        lanes_in_order();
    }
    update();
    put_row(n - 1);
    lanes_in_order();
    if (h == 0 && n > 1 && i == n - 2) d[n - 2] = x;
    if (h == 0 && i == n - 1) {
        if (n > 1) e[n - 2] = x;
        d[n - 1] = lds.column[tri_lane(n - 1)];
    }
}

// Eigenvalues of T below z (see svd_direct_values.hip): t holds (e_{i-1}^2, d_i), eights of them; and the last polynomial, value * 2^expo up to
// a factor that is the same for every z.
template <int EIGHTS>
__device__ inline int sturm_below(const doublex2 (&t)[8 * EIGHTS], double z, float& value, int& expo)
{
    double p0 = 0.0, p1 = 1.0;
    unsigned signs = 0;
    expo = 0;
#pragma unroll
    for (int i = 0; i < 8 * EIGHTS; ++i) {
        const double p2 = fma(t[i].y - z, p1, -(t[i].x * p0));
        p0 = p1;
        p1 = p2;
        signs = __builtin_amdgcn_alignbit(signs, hi32(p1), 31);
        if (i % 8 == 7) {
            // the larger of the two to [0.5, 1): 2^(1022 - E), E its exponent as it is stored
            const unsigned e = max(hi32(p0) & 0x7ff00000u, hi32(p1) & 0x7ff00000u);
            const double scale = mk64(0u, 0x7fd00000u - e);
            p0 *= scale;
            p1 *= scale;
            expo += (int)(e >> 20);
        }
    }
    value = (float)p1;
    return __popc(signs ^ (signs >> 1));
}

// What the first pass of the search leaves.
struct FirstPass { int below[ST], expo[ST]; float value[ST]; };

// All eigenvalues of T, descending, by the ST threads of the workgroup (all call): a first pass at ST points, then 16 points per
// eigenvalue and pass, until a cell is left: evenly spaced, or, once the interval is narrow, around where the polynomial is expected to be
// zero (see svd_direct_values.hip).  fine: where in its cell an eigenvalue is.  T (8 EIGHTS entries, in LDS) in registers.
// 18 columns: 10.8 thousand cycles, two waves on a SIMD; 11.2 with evenly spaced points and a binary search of the first pass, and without `fine`.
template <int EIGHTS>
__device__ inline void eigenvalues(const doublex2* in, int n, FirstPass& first, double* lam, double* fine)
{
    constexpr u64 CELLS = (LAM_MAX_BITS - LAM_MIN_BITS) >> LAM_STEP_BITS, SPAN = CELLS / ST;
    constexpr int LANES = ST / THIN_R, HALF = LANES / 2;
    const int tid = threadIdx.x, lane = tid & 63;
    doublex2 t[8 * EIGHTS];
#pragma unroll
    for (int i = 0; i < 8 * EIGHTS; ++i) t[i] = in[i];
    float value;
    int expo;
    first.below[tid] = sturm_below<EIGHTS>(t, cell_start(SPAN * tid), value, expo);
    first.value[tid] = value;
    first.expo[tid] = expo;
    __syncthreads();
    const int l = tid & (LANES - 1), base = lane & ~(LANES - 1), i = tid / LANES, asc = n - 1 - i;
    if (i < n) {
        const u64 group = ((1ull << LANES) - 1) << base;
        // last point with at most asc eigenvalues below it: of sixteen runs of 32, of sixteen pairs, of the two
        static_assert(ST == 2 * LANES * LANES, "three steps");
        auto held = [&](int at) { return __popcll(__ballot(first.below[at] <= asc) & group); };
        const int run = max(held(2 * LANES * l) - 1, 0) * 2 * LANES, pair = run + max(held(run + 2 * l) - 1, 0) * 2;
        const int lo = pair + (first.below[pair + 1] <= asc ? 1 : 0);
        const bool zero = first.below[0] > asc;
        const int hi = min(lo + 1, ST - 1);
        u64 g0 = SPAN * lo;
        unsigned width = zero ? 0u : (unsigned)SPAN;             // of the interval from g0 on
        // the polynomial at its ends, of the same sign as long as it is not known
        float f0 = first.value[lo], f1 = hi > lo ? first.value[hi] : f0;
        int e0 = first.expo[lo], e1 = first.expo[hi];
        static_assert(SPAN * LANES <= 0xffffffffull, "points of an interval in 32 bits");
        const int shift = 2 + 2 * (l < HALF ? l : LANES - 1 - l);
        bool uniform = false;
        while (width > 1) {                                      // (the lanes of an eigenvalue agree)
            unsigned point = width * (unsigned)(l + 1) / (unsigned)(LANES + 1);
            const bool near = !uniform && (f0 < 0.0f) != (f1 < 0.0f) && (u64)width * (unsigned)n < 1ull << (LAM_BITS - 4);
            if (near) {
                const float there = f0 * __builtin_amdgcn_rcpf(f0 - ldexpf(f1, e1 - e0));
                const unsigned at = min((unsigned)(there * (float)width), width - 1u), offset = width >> shift;
                point = min(max(l < HALF ? at - min(offset, at) : at + max(offset, 1u), 1u), width - 1u);
            }
            const int k = __popcll(__ballot(sturm_below<EIGHTS>(t, cell_start(g0 + point), value, expo) <= asc) & group);
            const int before = base + max(k - 1, 0), behind = base + min(k, LANES - 1);
            const unsigned p_lo = __shfl(point, before), p_hi = __shfl(point, behind);
            const float v_lo = __shfl(value, before), v_hi = __shfl(value, behind);
            const int x_lo = __shfl(expo, before), x_hi = __shfl(expo, behind);
            const unsigned from = k > 0 ? p_lo : 0u, to = k < LANES ? p_hi : width;
            if (k > 0) f0 = v_lo, e0 = x_lo;
            if (k < LANES) f1 = v_hi, e1 = x_hi;
            uniform = near && (u64)(to - from) * (unsigned)(LANES + 1) > width;  // (not there: eigenvalues too close to each other)
            g0 += from;
            width = to - from;
        }
        if (l == 0) {
            const u64 cell = LAM_MIN_BITS + (g0 << LAM_STEP_BITS), middle = 1ull << (LAM_STEP_BITS - 1);
            u64 inside = middle;
            if (width == 1u && (f0 < 0.0f) != (f1 < 0.0f)) {
                const double there = (double)f0 / ((double)f0 - ldexp((double)f1, e1 - e0));
                inside = min((u64)(there * (double)(1ull << LAM_STEP_BITS)), (1ull << LAM_STEP_BITS) - 1);
            }
            lam[i] = zero ? 0.0 : bits_double(cell + middle);
            fine[i] = zero ? 0.0 : bits_double(cell + inside);
        }
    }
}

template <int CTRL>
__device__ inline double dpp_or_one(double x)
{
    return mk64((unsigned)__builtin_amdgcn_update_dpp(0, (int)lo32(x), CTRL, 0xF, 0xF, false),
                (unsigned)__builtin_amdgcn_update_dpp(0x3FF00000, (int)hi32(x), CTRL, 0xF, 0xF, false));
}

// Unit eigenvector of T for the eigenvalue next to lam, by a wave: entry lane mod 32 in either half.  A twisted factorisation: the
// lower half of the lanes works out the pivots from the top, the upper half those from the bottom, as quotients of the
// characteristic polynomials (every lane runs through the recurrence and keeps its own step); the two are joined where they
// meet with the smallest pivot, and the entries are products of quotients from there, by scans.  The Rayleigh quotient
// corrects lam, for up to three rounds; one is enough as a rule, from where the eigenvalue is in its cell: if its residual is under `close`,
// which turns the vector by less than 1e-9, a sixtieth of a unit of fp32, and passes.  (Always three, from the middle of the cell: 15 thousand cycles.)
// t: as for sturm_below (n entries after the padding), e: off-diagonal.  good: of the residual |T z - lam z|; accepted: it passes.
__device__ inline double twisted_vector(const doublex2* t, const double* e, int n, double lam, double close, double good, const KeptApart& apart,
                                        bool& accepted)
{
    const int lane = threadIdx.x & 63, i = lane & 31;
    const bool bottom = lane >= 32;
    const double di = t[min(i, n - 1)].y;
    const double ei = i < n - 1 ? e[i] : 0.0, eb = i > 0 && i < n ? e[i - 1] : 0.0;
    double z = 0.0, inv = 1.0;
    for (int round = 0; round < 3; ++round) {
        double p0 = 0.0, p1 = 1.0, num = 1.0, den = 1.0;
        for (int k0 = 0; k0 < n; k0 += 8) {
            double d[8], off[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = min(k0 + u, n - 1);
                d[u] = t[bottom ? n - 1 - k : k].y;
                off[u] = k0 + u == 0 ? 0.0 : t[bottom ? n - k : k].x;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const double p2 = fma(d[u] - lam, p1, -(off[u] * p0));
                if (k0 + u == (bottom ? n - 1 - i : i)) { num = p2; den = p1; }
                p0 = p1;
                p1 = p2;
            }
            const int ex = max(__builtin_amdgcn_frexp_exp(p0), __builtin_amdgcn_frexp_exp(p1));
            p0 = __builtin_amdgcn_ldexp(p0, -ex);
            p1 = __builtin_amdgcn_ldexp(p1, -ex);
        }
        auto away_from_zero = [](double x) { return fabs(x) < 1e-290 ? copysign(1e-290, x) : x; };
        den = away_from_zero(den);
        num = away_from_zero(num);
        const double pivot = num * reciprocal(den);
        const double g = fold32(pivot, pivot) - (di - lam);
        // the smallest |g| of the entries there are, with its place in the lowest bits
        u64 least = i < n ? (((u64)__double_as_longlong(fabs(g))) & ~31ull) | (unsigned)i : ~0ull;
        auto smaller = [&](u64 o) { least = o < least ? o : least; };
        smaller((u64)__double_as_longlong(dpp<DPP_XOR1>(__longlong_as_double((long long)least))));
        smaller((u64)__double_as_longlong(dpp<DPP_XOR2>(__longlong_as_double((long long)least))));
        smaller((u64)__double_as_longlong(dpp<DPP_HALF_MIRROR>(__longlong_as_double((long long)least))));
        smaller((u64)__double_as_longlong(dpp<DPP_MIRROR>(__longlong_as_double((long long)least))));
        const double least_d = __longlong_as_double((long long)least);
        smaller((u64)__double_as_longlong(lane_value(least_d, 0)));
        smaller((u64)__double_as_longlong(lane_value(least_d, 16)));
        const int at = __builtin_amdgcn_readfirstlane((int)(least & 31ull));
        const double g_at = lane_value(g, at);
        // z_i = -(e_i / pivot_i) z_{i+1} above, -(e_{i-1} / pivot_i) z_{i-1} below
        const bool mine = bottom ? i > at && i < n : i < at;
        double f = mine ? -(bottom ? eb : ei) * (den * reciprocal(num)) : 1.0;
        auto step = [&](double shl, double shr) { f *= bottom ? shr : shl; };
        step(dpp_or_one<0x101>(f), dpp_or_one<0x111>(f));
        step(dpp_or_one<0x102>(f), dpp_or_one<0x112>(f));
        step(dpp_or_one<0x104>(f), dpp_or_one<0x114>(f));
        step(dpp_or_one<0x108>(f), dpp_or_one<0x118>(f));
        const double row1 = lane_value(f, 16), row2 = lane_value(f, 47);
        f *= lane < 16 ? row1 : lane >= 48 ? row2 : 1.0;
        const double own = mine ? f : !bottom && i == at ? 1.0 : 0.0;
        z = fold32(own, own);
        const double z2 = z * z;
        double sum = sum8(z2), weighted = sum8(z2 * (fabs(di) + (fabs(ei) + fabs(eb))));
        sum += dpp<DPP_MIRROR>(sum);
        weighted += dpp<DPP_MIRROR>(weighted);
        const double len2 = fold16(sum, sum);
        weighted = fold16(weighted, weighted);
        inv = inverse_root(len2);
        lam += g_at * (inv * inv);
        const double residual = fabs(g_at) * inv;
        accepted = residual <= good && apart.vector(residual, weighted * (inv * inv), lam);
        if (accepted && residual <= close) break;
    }
    return z * inv;
}

// Two ways to the spectrum.  The direct one, as for larger matrices (svd_direct.hip): tridiagonal form, Sturm counts, vectors of
// the kept atoms only.  It is accepted under the same conditions (the spectrum resolved down to four times the floor, rows of
// zeros aside; vectors with a small residual, kept ones apart); otherwise the two-sided Jacobi iteration.  18
// columns: 25 us; Jacobi in eight sweeps 73.  In thousands of cycles (2^16 positions): sums of the partial matrices 7, the reduction 20, eigenvalues 11,
// draw 1.6, vectors 6.5, back through the reflectors 3.7.  Before, 33 us: the trace entry by entry (2.2), the draw with a sum over the sigmas one
// after the other and its Philox rounds behind the spectrum (4.3), the header in front of the way back (2.4), always three rounds for a vector
// (15), one reflector at a time (5.2), all of 32 columns in the reduction (21.5).  T takes 96 of its 224 registers for 18 columns, 128 for 32: two waves on
// every SIMD do not fit beside a workgroup of the reduction of larger matrices (251 registers), and where those fill
// the chip it waits for the first of them to end.  That costs a call nothing, measured with a form of 158 registers, which did not fit either:
// the directly solved layers of ResNet-18 with its two thin ones 851 us, 852 with a form of 124 registers that fitted; with 256 chunks of
// positions 853 and 857, with 100 small matrices 859 and 860.
// Bound: latency.  Jacobi: one barrier per round of the tournament.  A is in two buffers: a round reads one and writes the other, one
// 2 x 2 block per thread; other threads rotate the vectors in place, two pairs of entries each.  Every wave works out all
// rotations of the round for itself and hands them around inside.
__global__ __launch_bounds__(ST) void thin_solve(const ThinMat* mats, double s, u64 seed, int* flags)
{
    __shared__ double A[2][THIN_R * LD], V[THIN_R * LD];         // direct: A[1] the matrix that is reduced, V the reflectors
    __shared__ doublex2 T[THIN_R];
    __shared__ double td[THIN_R], te[THIN_R], ttau[THIN_R], tw[THIN_R], pairs[THIN_R / 2];
    __shared__ __attribute__((aligned(16))) TriScratch tri;
    __shared__ FirstPass first;
    __shared__ int kept_at[THIN_R];
    __shared__ float uniform[THIN_R];
    __shared__ int unfinished[2];
    __shared__ double lam[THIN_R], fine[THIN_R];
    __shared__ int rank_of[THIN_R];
    __shared__ u64 drawn;
    __shared__ int accepted;
    const ThinMat& m = mats[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = m.r;
    // C in both triangles: sums over the chunks, of the entries i <= j that there are, in the order in which a partial sum holds
    // them (a wave's 64 entries are a few lines of memory: 128 partial sums 11 us with a line per entry, 4.7 so).  Up to 256 of
    // them leave half of the threads for the second half of the chunks.
    {
        const int entries = r * (r + 1) / 2, parts = entries <= ST / 2 ? 2 : 1;
        const int share = (m.nchunks + parts - 1) / parts;
        for (int f = tid & (ST / parts - 1); f < entries; f += ST / parts) {
            // f = j (j + 1) / 2 + i
            int j = (int)((sqrtf(8.0f * (float)f + 1.0f) - 1.0f) * 0.5f);
            j += (j + 1) * (j + 2) / 2 <= f;
            j -= j * (j + 1) / 2 > f;
            const int i = f - j * (j + 1) / 2;
            const int e = j < 16 ? j * 16 + i : i < 16 ? 256 + (j - 16) * 16 + i : 512 + (j - 16) * 16 + i - 16;
            const Global<const double> in = global((const double*)m.part) + e;
            const int part = tid / (ST / parts);
            int c = part * share;
            const int end = min(m.nchunks, c + share);
            double sum = 0.0;
            for (; c + 32 <= end; c += 32) {
                double x[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) x[u] = in[(size_t)(c + u) * PART];
#pragma unroll
                for (int u = 0; u < 32; ++u) sum += x[u];
            }
            for (; c < end; c += 8) {
                double x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = in[(size_t)min(c + u, end - 1) * PART];
#pragma unroll
                for (int u = 0; u < 8; ++u) sum += c + u < end ? x[u] : 0.0;
            }
            A[part][i * LD + j] = sum;
        }
        __syncthreads();
        for (int e = tid; e < r * THIN_R; e += ST) {
            const int i = e >> 5, j = e & 31;
            if (i <= j && j < r) {
                const double sum = A[0][i * LD + j] + (parts == 2 ? A[1][i * LD + j] : 0.0);
                A[0][i * LD + j] = sum;
                A[0][j * LD + i] = sum;
            }
        }
    }
    if (tid < 2) unfinished[tid] = 0;
    __syncthreads();
    const double own_norm = A[0][min(lane, r - 1) * (LD + 1)], trace = wave_sum(lane < r ? own_norm : 0.0);
    const int zero_rows = __popcll(__ballot(lane < r && own_norm == 0.0));
    // wave 0: sigma, Algorithm 1 (the first index whose probability stays under 1, see block_algorithm1), the draw
    float sigma = 0.0f, p = 0.0f;
    u64 mask = 0ull;
    auto draw = [&] {
        const double l0 = lam[rank_of[0]];
        const double l = lam[lane < r ? rank_of[lane] : 0];
        const bool real = lane < r && l > (double)svd::ZERO_REL * l0;
        sigma = real ? (float)sqrt(l) : 0.0f;
        double tail = (double)sigma;                             // sum of the sigmas from this one on (exact: 47 bits)
        tail += dpp<DPP_SHL1>(tail);
        tail += dpp<DPP_SHL2>(tail);
        tail += dpp<DPP_SHL4>(tail);
        tail += dpp<DPP_SHL8>(tail);
        static_assert(THIN_R == 32, "two rows of lanes");
        tail += lane < 16 ? lane_value(tail, 16) : 0.0;
        const u64 under = __ballot(lane < r && (double)sigma * (s - (double)lane) <= tail);
        const int ns = under ? __ffsll((unsigned long long)under) - 1 : r;
        const double tail_ns = ns < r ? __shfl(tail, ns) : 0.0;
        p = lane < r ? alg1_probability(sigma, lane, ns, s, tail_ns) : 0.0f;
        mask = __ballot(lane < r && uniform[min(lane, r - 1)] < p);
    };
    // ... of which nothing but the comparison needs the spectrum
    auto uniforms = [&] {
        if (lane < THIN_R) {
            const u32x4 rnd = philox4x32_10((u64)(lane >> 2), m.stream_id, seed);
            const uint32_t word = (lane & 3) == 0 ? rnd.x : (lane & 3) == 1 ? rnd.y : (lane & 3) == 2 ? rnd.z : rnd.w;
            uniform[lane] = u01(word);
        }
    };
    // wave 0: what the other waves have to know of the kept atoms; sigma in the scale of the data
    auto list_kept = [&] {
        const int pos = __popcll(mask & ((1ull << lane) - 1));
        if ((mask >> lane) & 1ull) {
            kept_at[pos] = lane;
            tw[pos] = sigma / p;
        }
        if (lane == 0) drawn = mask;
    };
    bool direct = trace > 1e-280 && trace < 1e280;               // (false for NaN)
    int expo = 0;
    if (direct) {
        // scaled by a power of four to a trace in [1/4, 1)
        (void)frexp(trace, &expo);
        expo += expo & 1;
        for (int e = tid; e < THIN_R * LD; e += ST) {
            const int i = e / LD, j = e - i * LD;
            A[1][e] = i < r && j < r ? ldexp(A[0][e], -expo) : 0.0;
        }
        __syncthreads();
        if (wave == 0) {
            if (r <= 8) tridiagonal<4>(A[1], V, tri, td, te, ttau, r);
            else if (r <= 16) tridiagonal<8>(A[1], V, tri, td, te, ttau, r);
            else if (r <= 20) tridiagonal<10>(A[1], V, tri, td, te, ttau, r);
            else tridiagonal<16>(A[1], V, tri, td, te, ttau, r);
        }
        if (wave == 1) uniforms();
        __syncthreads();
        const int n_pad = (r + 7) & ~7, pad = n_pad - r;
        if (tid < n_pad) {
            const int i = tid - pad;
            const double off = i > 0 ? te[i - 1] : 0.0;
            T[tid] = i < 0 ? doublex2{0.0, 2.0} : doublex2{i > 0 ? fmax(off * off, OD2_MIN) : 0.0, td[i]};
        }
        if (tid < THIN_R) rank_of[tid] = tid;
        __syncthreads();
        if (n_pad == 8) eigenvalues<1>(T, r, first, lam, fine);
        else if (n_pad == 16) eigenvalues<2>(T, r, first, lam, fine);
        else if (n_pad == 24) eigenvalues<3>(T, r, first, lam, fine);
        else eigenvalues<4>(T, r, first, lam, fine);
        __syncthreads();
        if (wave == 0) {
            draw();
            const bool resolved = zero_rows >= r || lam[r - 1 - zero_rows] > FLOOR_REL * lam[0];
            if (lane == 0) accepted = resolved;
            sigma = (float)ldexp((double)sigma, expo / 2);
            list_kept();
        } else {
            // products of the neighbouring reflectors that are applied together
            for (int q = wave - 1; q < (r - 2) / 2; q += ST / 64 - 1) {
                const int k = r - 3 - 2 * q;
                const double product = wave_sum(lane < THIN_R ? V[k * LD + lane] * V[(k - 1) * LD + lane] : 0.0);
                if (lane == 0) pairs[q] = product;
            }
        }
        __syncthreads();
        const int count = accepted ? min(__popcll(drawn), m.capacity) : 0;
        for (int a = wave; a < count; a += ST / 64) {
            const int at = kept_at[a];
            const double own = lam[at], gap = fmin(at > 0 ? lam[at - 1] - own : 1e300, at + 1 < r ? own - lam[at + 1] : 1e300);
            // (2^-22: from a distance of that the three rounds end with vectors apart)
            const KeptApart apart(own, a > 0 ? lam[kept_at[a - 1]] : -1.0, a + 1 < count ? lam[kept_at[a + 1]] : -1.0,
                                  2.384185791015625e-07);
            bool good = false;
            const double z = twisted_vector(T + pad, te, r, fine[at], 1e-9 * gap, 1e-12 * lam[0], apart, good);
            if (lane < THIN_R) A[1][a * LD + lane] = z;
            if (lane == 0 && !good) accepted = 0;
        }
        __syncthreads();
        direct = accepted != 0;
    }
    bool open = false;
    if (!direct) {
        for (int e = tid; e < THIN_R * THIN_R; e += ST) V[(e >> 5) * LD + (e & 31)] = (e >> 5) == (e & 31) ? 1.0 : 0.0;
        if (wave == 1) uniforms();
        __syncthreads();
        // tournament over n = r rounded up to even (an entry past r is a row of zeros and never rotates)
        const int n = (r + 1) & ~1, half = n >> 1, n1 = n - 1;
        if (r & 1) {                                                 // the row and column of zeros
            __syncthreads();
            if (tid < n) A[0][r * LD + tid] = A[0][tid * LD + r] = 0.0;
            __syncthreads();
        }
        // half^2 blocks of A on the first waves, as many pairs of entries of V (rows ka and ka + half) on the next ones: four waves,
        // one per SIMD, up to 22 vectors
        const int waves = (half * half + 63) >> 6, role = wave / waves;         // 0: A, 1: V, above: no part in it
        const int first_e = (wave - role * waves) << 6, item = first_e + lane;
        const int ka = item / half, kb = item - ka * half;
        const bool valid = item < half * half;
        const int lane_a = min(ka, half - 1) - first_e % half;                  // lane whose pair kb is pair ka
        const int src_a = lane_a < 0 ? lane_a + half : lane_a;
        const double floor = 1e-13 * trace;
        // round t pairs n1 with t and t + k with t - k (mod n1); a thread holds pairs ka and kb and moves them on by one per round
        auto first_of = [&](int k, int& p, int& q) {
            p = k == 0 ? n1 : k;
            q = k == 0 ? 0 : n1 - k;
        };
        auto move_on = [&](int k, int& p, int& q) {
            if (k != 0) p = p + 1 == n1 ? 0 : p + 1;
            q = q + 1 == n1 ? 0 : q + 1;
        };
        auto at = [](int i) { return (i << 5) + i; };                // i * LD
        static_assert(LD == 33, "row offsets by shift and add");
        const int row_v = at(min(ka, half - 1)), row_w = row_v + at(half);
        int pa, qa, pb, qb;
        first_of(min(ka, half - 1), pa, qa);
        first_of(kb, pb, qb);
        int cur = 0, sweeps = 0;
        open = n > 1 && trace > 0.0;
        while (open && sweeps < MAX_SWEEPS) {
            bool turned = false;
            for (int round = 0; round < n1; ++round) {
                if (role < 2) {
                    const double* old = A[cur];
                    double* now = A[cur ^ 1];
                    // everything that will be needed, on its way before the rotations
                    const int ra = at(pa), sa_ = at(qa), rb = at(pb), sb_ = at(qb);
                    const double dp = old[rb + pb], dq = old[sb_ + qb], g = old[rb + qb];
                    const double* from = role == 0 ? old : V;
                    const int up = role == 0 ? ra : row_v, down = role == 0 ? sa_ : row_w;
                    const double b00 = from[up + pb], b01 = from[up + qb], b10 = from[down + pb], b11 = from[down + qb];
                    double cb, sb;
                    rotation(dp, dq, g, cb, sb);
                    // the sweep is the last one if all cosines it met were small (what it leaves is then their square), rows at
                    // the rounding of the largest aside
                    turned = turned || (g * g > 1e-12 * dp * dq && fmin(dp, dq) > floor);
                    const double c00 = cb * b00 - sb * b01, c01 = sb * b00 + cb * b01;
                    const double c10 = cb * b10 - sb * b11, c11 = sb * b10 + cb * b11;
                    if (role == 0) {
                        const double ca = __shfl(cb, src_a), sa = __shfl(sb, src_a);
                        if (valid) {
                            const bool diagonal = ka == kb;
                            now[ra + pb] = ca * c00 - sa * c10;
                            now[ra + qb] = diagonal ? 0.0 : ca * c01 - sa * c11;
                            now[sa_ + pb] = diagonal ? 0.0 : sa * c00 + ca * c10;
                            now[sa_ + qb] = sa * c01 + ca * c11;
                        }
                    } else if (valid) {
                        V[up + pb] = c00;
                        V[up + qb] = c01;
                        V[down + pb] = c10;
                        V[down + qb] = c11;
                    }
                    move_on(ka, pa, qa);
                    move_on(kb, pb, qb);
                }
                __syncthreads();
                cur ^= 1;
            }
            if (turned) unfinished[sweeps & 1] = 1;
            __syncthreads();
            open = unfinished[sweeps & 1] != 0;
            ++sweeps;
            if (tid == 0) unfinished[sweeps & 1] = 0;                // (written again only after the barriers of the next sweep)
        }
        if (tid < r) lam[tid] = A[cur][tid * LD + tid];
        if (tid < THIN_R) rank_of[tid] = 0;                          // (not all of them are written if lam is not a number)
        __syncthreads();
        if (tid < r) {
            int before = 0;
            const double mine = lam[tid];
            for (int j = 0; j < r; ++j) before += lam[j] > mine || (lam[j] == mine && j < tid);
            rank_of[before] = tid;
        }
        __syncthreads();
        if (wave == 0) {
            draw();
            list_kept();
        }
        __syncthreads();
    }
    // header by wave 0; the kept vectors, one wave each, from wave 1 on
    if (wave == 0) {
        if (lane < r) {
            if (m.sigma_out) m.sigma_out[lane] = sigma;
            if (m.p_out) m.p_out[lane] = p;
        }
        if (lane == 0) {
            *m.count = __popcll(mask);
            m.report[0] = 1;
            m.report[1] = 2;
            atomicMax(&flags[FLAG_MAX_SWEEPS], 1);
            if (__popcll(mask) > m.capacity) atomicMax(&flags[FLAG_CAPACITY], 1);
            if (open && !(trace != trace)) atomicMax(&flags[FLAG_NOCONV], 1);
        }
        const int pos = __popcll(mask & ((1ull << lane) - 1));
        if (((mask >> lane) & 1ull) && pos < m.capacity) {
            m.idx[pos] = lane;
            if (m.w) m.w[pos] = sigma / p;
        }
    }
    const int count = min(__popcll(drawn), m.capacity);
    for (int a = (wave + ST / 64 - 1) % (ST / 64); a < count; a += ST / 64) {
        const int i = lane & 31, src = rank_of[kept_at[a]];
        double x, inv = inverse_root(lam[src]);
        if (direct) {
            // H z, the last step's reflection first, two at a time: both products with z in one sum, one in each half of the lanes
            x = i < r ? A[1][a * LD + i] : 0.0;
            int k = r - 3;
            for (int q = 0; k > 0; k -= 2, ++q) {
                const double v = V[k * LD + i], u = V[(k - 1) * LD + i];
                double sum = sum8((lane < 32 ? v : u) * x);
                sum += dpp<DPP_MIRROR>(sum);
                sum = fold16(sum, sum);
                const double tv = ttau[k] * lane_value(sum, 0);
                const double tu = ttau[k - 1] * fma(-tv, pairs[q], lane_value(sum, 32));
                x = fma(-tu, u, fma(-tv, v, x));
            }
            if (k == 0) x = fma(-ttau[0] * wave_sum(lane < 32 ? V[i] * x : 0.0), V[i], x);
            inv = ldexp(inv, -(expo / 2));
        } else {
            x = i < r ? V[i * LD + src] : 0.0;
        }
        const double fold = m.w ? 1.0 : (double)tw[a];           // folded message: the weight goes into U
        if (lane < r) {
            global(m.tall ? m.V + (size_t)a * r : m.U + (size_t)a * r)[i] = (float)(m.tall ? x : x * fold);
            global(m.u)[a * r + i] = x * inv * (m.tall ? fold : 1.0);
        }
    }
}

// ------------------------------------------------------------------------------------------------
constexpr int LONG_POS = 256;                  // positions per workgroup, one per thread
constexpr int LONG_GROUP = 8;

// acc[k] += x * u[k][i], the u by scalar loads (the same for all lanes)
template <int NK>
__device__ inline void long_dots(const float* mine /* LDS, r entries */, const __attribute__((address_space(4))) double* u, int r,
                                 double (&acc)[LONG_GROUP])
{
    for (int i = 0; i < r; ++i) {
        const double d = (double)mine[i];
#pragma unroll
        for (int k = 0; k < NK; ++k) acc[k] = fma(d, u[k * r + i], acc[k]);
    }
}

// Bound: one read of the data; 11.16 M elements of 18 columns in 14 us (15 with LDS for 32 columns whatever their number, which
// leaves room for four workgroups per compute unit instead of eight; 34 with four dependent rounds of loads per workgroup and the
// atoms in LDS).  The entries of a block of positions are fetched before anything is known about the kept atoms,
// go through LDS (those of a position of a tall matrix lie side by side, and a thread owns a position) and are multiplied with up
// to eight atoms per pass.
__global__ __launch_bounds__(LONG_POS) void thin_long(const ThinMat* mats, const Work* work)
{
    extern __shared__ float xs[];                                // [LONG_POS][r | 1]
    const Work wk = work[blockIdx.x];
    const ThinMat& m = mats[wk.mat];
    const int r = m.r, tid = threadIdx.x;
    const bool tall = m.tall;
    const Global<const float> G = global(m.G);
    const int ls = r | 1;                                        // stride of a position in LDS
    const int by_r = ((1 << 20) + r - 1) / r;
    const int first = wk.a * LONG_POS, here = min(LONG_POS, m.M - first);
    if (tall) {
        const Global<const float> block = G + (long long)first * m.ldg;
        const int total = here * r;
        // element e of the block: position e / r (by a multiplication that is exact below 2^13), entry e mod r
        auto put = [&](int e, float x) {
            const int p = (e * by_r) >> 20;
            xs[p * ls + (e - p * r)] = x;
        };
        if (m.ldg == r && (((size_t)m.G) & 15) == 0) {           // (a block is a multiple of 16 bytes long)
            typedef float floatx4 __attribute__((ext_vector_type(4)));
            const Global<const floatx4> quads = (Global<const floatx4>)block;
            floatx4 x[THIN_R / 4];
#pragma unroll
            for (int u = 0; u < THIN_R / 4; ++u)
                if ((tid + LONG_POS * u) * 4 + 3 < total) x[u] = quads[tid + LONG_POS * u];
#pragma unroll
            for (int u = 0; u < THIN_R / 4; ++u) {
                const int e = (tid + LONG_POS * u) * 4;
                if (e + 3 < total) {
                    put(e, x[u].x);
                    put(e + 1, x[u].y);
                    put(e + 2, x[u].z);
                    put(e + 3, x[u].w);
                }
            }
            if (tid < (total & 3)) put((total & ~3) + tid, block[(total & ~3) + tid]);
        } else {
            for (int e0 = tid; e0 < total; e0 += 8 * LONG_POS) {
                float x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = min(e0 + LONG_POS * u, total - 1), p = (e * by_r) >> 20;
                    x[u] = block[(long long)p * m.ldg + (e - p * r)];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) put(min(e0 + LONG_POS * u, total - 1), x[u]);
            }
        }
    } else {
        const Global<const float> g = G + first + min(tid, here - 1);
        for (int i0 = 0; i0 < r; i0 += 16) {
            float x[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) x[u] = g[min(i0 + u, r - 1) * m.ldg];
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (i0 + u < r) xs[tid * ls + i0 + u] = x[u];
        }
    }
    const int kept = min(*m.count, m.capacity);
    __syncthreads();
    if (tid >= here) return;
    const Global<float> out = global(tall ? m.U : m.V) + first + tid;
    const float* mine = xs + tid * ls;
    for (int s0 = 0; s0 < kept; s0 += LONG_GROUP) {
        const int ns = min(LONG_GROUP, kept - s0);
        const __attribute__((address_space(4))) double* u = (const __attribute__((address_space(4))) double*)(m.u + s0 * r);
        double acc[LONG_GROUP] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        if (ns <= 2) long_dots<2>(mine, u, r, acc);              // (a vector past the kept ones is read but not used)
        else if (ns <= 4) long_dots<4>(mine, u, r, acc);
        else long_dots<8>(mine, u, r, acc);
#pragma unroll
        for (int k = 0; k < LONG_GROUP; ++k)
            if (k < ns) out[(size_t)(s0 + k) * m.M] = (float)acc[k];
    }
}

}  // namespace

void plan_matrix(Carver& carve, ThinMat& m)
{
    // chunks of GRAM_CHUNK positions, larger only to keep a matrix under 128 of them; from the shape alone, so that the sums do not
    // depend on what else is in the call
    const long long runs = ((long long)m.M + GRAM_CHUNK - 1) / GRAM_CHUNK;
    m.chunk = (int)(GRAM_CHUNK * ((runs + MAX_CHUNKS - 1) / MAX_CHUNKS));
    m.nchunks = (int)(((long long)m.M + m.chunk - 1) / m.chunk);
    m.part = carve.take<double>((size_t)m.nchunks * PART);
    m.u = carve.take<double>((size_t)(m.r + LONG_GROUP) * m.r);          // (thin_long reads whole groups)
}

void plan_work(ThinPlan& plan)
{
    for (size_t j = 0; j < plan.mats.size(); ++j) {
        const ThinMat& m = plan.mats[j];
        for (int c = 0; c < m.nchunks; ++c) plan.gram.push_back(Work{(int)j, c, 0, 0});
        for (int c = 0; c < (m.M + LONG_POS - 1) / LONG_POS; ++c) plan.lng.push_back(Work{(int)j, c, 0, 0});
    }
}

hipError_t launch(const ThinPlan& plan, const ThinMat* d_mats, const Work* gram, const Work* lng, double s, uint64_t seed, int* d_flags,
                  hipStream_t stream, hipEvent_t done)
{
    thin_gram<<<(unsigned)plan.gram.size(), 64 * GRAM_WAVES, 0, stream>>>(d_mats, gram);
    thin_solve<<<(unsigned)plan.mats.size(), ST, 0, stream>>>(d_mats, s, (u64)seed, d_flags);
    int most = 0;
    for (const ThinMat& m : plan.mats) most = std::max(most, m.r | 1);
    return launch_recorded(done, thin_long, (unsigned)plan.lng.size(), LONG_POS, LONG_POS * most * sizeof(float), stream, d_mats, lng);
}

}  // namespace thin
}  // namespace atomo
