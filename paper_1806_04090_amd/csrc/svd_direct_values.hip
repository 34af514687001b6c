// Direct Spectral-ATOMO encode: all eigenvalues of the tridiagonal matrices by multisection with Sturm counts, and the factors of the
// blocks of reflectors, in one launch.
//
// A file of its own for its compiler flags: the loops of svd_direct.hip are aligned, for the steps of the reduction, and the search takes
// longer if its own are (the ResNet-18 layers 55.9 us where the compiler puts them, 57.8 at 64 bytes).
#include "svd_device.h"
#include "svd_direct.h"

namespace atomo {
namespace direct {

using svd::Work;

namespace {

// ------------------------------------------------------------------------------------------------
// Blocks of reflectors
// ------------------------------------------------------------------------------------------------
// H = H_0 H_1 .. in blocks of 16 reflectors, each I - V F V^T with V the 16 vectors and F upper triangular: column i of F is
// -tau_i F (V^T v_i) above the diagonal and tau_i on it.  One workgroup per block: the 16 x 16 products V^T V on the
// matrix cores (every wave a quarter of the columns), then the columns of F one after the other.
__device__ inline void block_factor(const DirectMat& m, int b)
{
    __shared__ double gram[4][RB][RB + 1], f[RB][RB + 1], tau[RB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, q = lane >> 4;
    const int N = m.nt * TILE, k0 = b * RB, k = k0 + l16;
    const bool live = k >= m.pad && k < N - 2;
    const Global<const double> row = global((const double*)m.refl) + (size_t)k * N;
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int c = (k0 & ~63) + 16 * wave; c < N; c += 64) {
        doublex2 v[2] = {doublex2{0.0, 0.0}, doublex2{0.0, 0.0}};
        if (live) {
            v[0] = *(Global<const doublex2>)(row + c + 4 * q);
            v[1] = *(Global<const doublex2>)(row + c + 4 * q + 2);
        }
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[0].x, v[0].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[0].y, v[0].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[1].x, v[1].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[1].y, v[1].y, acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) gram[wave][4 * v + q][l16] = acc[v];
    if (tid < RB) tau[tid] = live ? m.tau[k] : 0.0;
    __syncthreads();
    gram[0][tid >> 4][tid & 15] = (gram[0][tid >> 4][tid & 15] + gram[1][tid >> 4][tid & 15]) +
                                  (gram[2][tid >> 4][tid & 15] + gram[3][tid >> 4][tid & 15]);
    __syncthreads();
    if (tid < RB) {                                              // thread r: row r of F
        double row_f[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            double sum = 0.0;
#pragma unroll
            for (int j = 0; j < i; ++j) sum = fma(row_f[j], gram[0][j][i], sum);
            row_f[i] = tid == i ? tau[i] : tid < i ? -tau[i] * sum : 0.0;
        }
#pragma unroll
        for (int i = 0; i < RB; ++i) f[tid][i] = row_f[i];
    }
    __syncthreads();
    m.fact[(size_t)b * (RB * RB) + tid] = f[tid >> 4][tid & 15];
}

// ------------------------------------------------------------------------------------------------
// Eigenvalues of T
// ------------------------------------------------------------------------------------------------
// How many eigenvalues of T lie below z: sign changes of the characteristic polynomials of the leading blocks,
// p_{i+1} = (d_i - z) p_i - e_{i-1}^2 p_{i-1} (no division; rescaled by a power of two every eight steps, the squared
// off-diagonals are kept above 2^-110 so that eight steps stay inside the range).  T comes through scalar loads, eight
// entries (e_{i-1}^2, d_i) at a time, the next eight on their way while these are worked on; the padding in front, (0, 2), leaves the
// sign as it is.
// Bound: issue, four instructions per step and ten per eight, 34 cycles per step with one wave on a SIMD (the entries from LDS, or the
// instructions of two steps interleaved: the same).
typedef unsigned uintx16 __attribute__((ext_vector_type(16)));
typedef const uintx16 __attribute__((address_space(4)))* scalar_ptr;   // read through the scalar cache, never written here

template <bool VALUE>
__device__ inline void sturm_steps(const uintx16& a, const uintx16& b, double z, double& p0, double& p1, unsigned& signs, int& expo)
{
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const uintx16& w = u < 4 ? a : b;
        const int x = 4 * (u & 3);
        const double p2 = fma(mk64(w[x + 2], w[x + 3]) - z, p1, -(mk64(w[x], w[x + 1]) * p0));
        p0 = p1;
        p1 = p2;
        signs = __builtin_amdgcn_alignbit(signs, hi32(p1), 31);
    }
    // the larger of the two to [0.5, 1): 2^(1022 - E), E its exponent as it is stored
    const unsigned e = max(hi32(p0) & 0x7ff00000u, hi32(p1) & 0x7ff00000u);
    const double scale = mk64(0u, 0x7fd00000u - e);
    p0 *= scale;
    p1 *= scale;
    if (VALUE) expo += (int)(e >> 20);
}
// a0, a1: the first entries of T, asked for; they are again when it returns.  VALUE: and the last polynomial, value * 2^expo up to a
// factor that is the same for every z.
struct Sturm {
    scalar_ptr t;
    int n;
    uintx16 a0, a1;
    __device__ inline Sturm(scalar_ptr entries, int count) : t(entries), n(count), a0(entries[0]), a1(entries[1]) {}
    template <bool VALUE>
    __device__ inline int below(double z, float& value, int& expo)
    {
        double p0 = 0.0, p1 = 1.0;
        int count = 0;
        expo = 0;
        unsigned signs = 0;
        for (int i = 0; i < n; i += 16) {
            // (a wait for scalar loads is one for all of them: the next go out behind it)
            asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(a0), "+s"(a1));
            uintx16 b0 = t[i / 4 + 2], b1 = t[i / 4 + 3];
            __builtin_amdgcn_sched_barrier(0);
            sturm_steps<VALUE>(a0, a1, z, p0, p1, signs, expo);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(b0), "+s"(b1));
            const int next = i + 16 < n ? i / 4 + 4 : 0;
            a0 = t[next];
            a1 = t[next + 1];
            __builtin_amdgcn_sched_barrier(0);
            sturm_steps<VALUE>(b0, b1, z, p0, p1, signs, expo);
            count += __popc((signs ^ (signs >> 1)) & 0xffffu);
            __builtin_amdgcn_sched_barrier(0);
        }
        value = (float)p1;
        return count;
    }
};

// Eigenvalue number i (descending) in [2^-50, 1), searched on the bit pattern of the double, in cells of 2^25 patterns
// (LAM_BITS relative bits): a first pass at 256 points and, if they are not far apart, a second one at 256 points between them for all
// eigenvalues of the workgroup, which are neighbours; then `lanes` points per eigenvalue and pass.  These are evenly spaced until
// the interval is 1 / (16 r) of the eigenvalue wide.  From there on the polynomial, which changes its sign in it, is nearly a line
// unless another eigenvalue is close: the points close in on where the line is zero by powers of two, and if the interval has
// not become smaller by as much as with evenly spaced ones, the next pass has those.  The counts alone decide: the cell that is found
// does not depend on how many points a pass has or where they are.
// Passes of a wave by 16 lanes for r = 512: 7.5 on average, 8 at most -> 5.1, 7; by four 12 -> 7.4.  The ResNet-18 layers 63.8 -> 55.2 us,
// 64 x (512 x 4608) 150 -> 111, 64 x 576 9.3 -> 9.3.
// Work: matrix, first eigenvalue; 256 / lanes eigenvalues per workgroup.  Behind the n_eig of these: matrix, block of
// reflectors (block_factor: wanted by the next kernels, and this one leaves the room).
__global__ __launch_bounds__(256) void direct_eigenvalues(const DirectMat* mats, const Work* work, int n_eig, int lanes)
{
    if ((int)blockIdx.x >= n_eig) {
        const Work wb = work[blockIdx.x];
        block_factor(mats[wb.mat], wb.a);
        return;
    }
    __shared__ int below[2][256];
    __shared__ float values[256];
    __shared__ int expos[256];
    constexpr u64 CELLS = (LAM_MAX_BITS - LAM_MIN_BITS) >> LAM_STEP_BITS, SPAN = CELLS / 256;
    const Work wk = work[blockIdx.x];
    const DirectMat& m = mats[wk.mat];
    const int tid = threadIdx.x, lane = tid & 63, n = m.r;
    const int first = m.pad & ~15;
    Sturm sturm((scalar_ptr)(u64)(m.td + first), m.nt * TILE - first);
    float value;
    int expo;
    below[0][tid] = sturm.below<false>(cell_start(SPAN * tid), value, expo);
    __syncthreads();
    const int l = tid & (lanes - 1), base = lane & ~(lanes - 1);
    const int i = min(wk.a + tid / lanes, n - 1);                // (a group past the end repeats the last one)
    const int asc = n - 1 - i;
    // last of 256 points with at most `most` eigenvalues below it
    auto last_point = [&](const int (&count)[256], int most) {
        int lo = 0;
#pragma unroll
        for (int half = 128; half > 0; half >>= 1) lo += count[lo + half] <= most ? half : 0;
        return lo;
    };
    const int lo = last_point(below[0], asc);
    const bool zero = below[0][0] > asc;
    // the interval: cells start + [r0, r1), and the polynomial at its ends, of the same sign as long as it is not known
    u64 start = SPAN * lo;
    unsigned r0 = 0u, r1 = zero ? 0u : (unsigned)SPAN;
    float f0 = 1.0f, f1 = 1.0f;
    int e0 = 0, e1 = 0;
    // the eigenvalues of the workgroup are neighbours: the second pass is at 256 points for all of them as well, if they are close
    const int from = last_point(below[0], n - 1 - min(wk.a + 256 / lanes - 1, n - 1)), to = last_point(below[0], n - 1 - wk.a);
    if ((to - from + 1) * (lanes + 1) < 256) {
        const unsigned step = (unsigned)(SPAN * (to - from + 1) / 256) + 1u;
        below[1][tid] = sturm.below<true>(cell_start(min(SPAN * from + (u64)(step * tid), CELLS)), value, expo);
        values[tid] = value;
        expos[tid] = expo;
        __syncthreads();
        if (!zero) {
            const int k = last_point(below[1], asc), k1 = min(k + 1, 255);
            start = SPAN * from;
            r0 = step * k;
            r1 = r0 + step;
            f0 = values[k], e0 = expos[k];
            f1 = k < 255 ? values[k1] : f0, e1 = expos[k1];
        }
    }
    const u64 group = ((1ull << lanes) - 1) << base;
    const float part = (float)(l + 1) / (float)(lanes + 1);
    // offsets from where the polynomial is expected to be zero: 2^-shift of the interval
    const int half = lanes / 2, number = l < half ? l : lanes - 1 - l;
    const int shift = 2 + (half == 2) + number * (half == 2 ? 5 : half == 4 ? 3 : half == 8 ? 2 : 1);
    bool uniform = false;
    while (!__all(r1 - r0 <= 1u)) {
        const unsigned width = r1 - r0;
        unsigned r = r0 + min((unsigned)((float)width * part), width);
        const bool near = !uniform && (f0 < 0.0f) != (f1 < 0.0f) && width > 1u && (u64)width * (unsigned)n < 1ull << (LAM_BITS - 4);
        if (near) {
            const float there = f0 * __builtin_amdgcn_rcpf(f0 - ldexpf(f1, e1 - e0));
            const unsigned at = min((unsigned)(there * (float)width), width - 1u), offset = width >> shift;
            r = r0 + min(max(l < half ? at - min(offset, at) : at + max(offset, 1u), 1u), width - 1u);
        }
        // points with at most asc eigenvalues below
        const int k = __popcll(__ballot(sturm.below<true>(cell_start(start + r), value, expo) <= asc) & group);
        const int before = base + max(k - 1, 0), behind = base + min(k, lanes - 1);
        const unsigned r_lo = __shfl(r, before), r_hi = __shfl(r, behind);
        const float v_lo = __shfl(value, before), v_hi = __shfl(value, behind);
        const int e_lo = __shfl(expo, before), e_hi = __shfl(expo, behind);
        if (k > 0) r0 = r_lo, f0 = v_lo, e0 = e_lo;
        if (k < lanes) r1 = r_hi, f1 = v_hi, e1 = e_hi;
        uniform = near && (u64)(r1 - r0) * (unsigned)(lanes + 1) > width;        // (not there: eigenvalues too close to each other)
    }
    // The polynomial at the ends of the cell says where in it the eigenvalue is (direct_vectors starts from there), to about 2^-20 of
    // the cell where others are far; lam itself stays the middle.
    const u64 cell = LAM_MIN_BITS + ((start + r0) << LAM_STEP_BITS), middle = 1ull << (LAM_STEP_BITS - 1);
    if (l == 0) {
        u64 inside = middle;
        if (r1 - r0 == 1u && (f0 < 0.0f) != (f1 < 0.0f)) {
            const double there = (double)f0 / ((double)f0 - ldexp((double)f1, e1 - e0));
            inside = min((u64)(there * (double)(1ull << LAM_STEP_BITS)), (1ull << LAM_STEP_BITS) - 1);
        }
        m.lam[i] = zero ? 0.0 : bits_double(cell + middle);
        m.fine[i] = zero ? 0.0 : bits_double(cell + inside);
    }
}

}  // namespace

void launch_eigenvalues(const DirectPlan& plan, const DirectTables& t, hipStream_t stream)
{
    direct_eigenvalues<<<(unsigned)plan.eig.size(), 256, 0, stream>>>(t.mats, t.eig, (int)plan.n_eig, plan.eig_lanes);
}

}  // namespace direct
}  // namespace atomo
