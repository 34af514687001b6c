// Spectral-ATOMO encode without an iteration over the data: Gram matrix in double precision, Householder reduction to
// tridiagonal form, all eigenvalues by multisection with Sturm counts, eigenvectors of the kept atoms only.
//
// A message holds about s atoms of r, but its probabilities need every singular value.  A Jacobi iteration computes all
// r singular pairs to get there.  Here the r x r matrix C = A A^T (A: the r vectors of the shorter side) is formed once,
// C = H T H^T with T tridiagonal, sigma_i = sqrt(lambda_i(T)), and after the Bernoulli draw only the kept atoms get an
// eigenvector of T, its image under H, and one product with the data for the other side.
//
// Precision.  Squaring loses half of the digits, so everything between the data and sigma is in double precision:
// products of two floats are exact there, lambda has an absolute error of about 1e-15 lambda_1, and sigma one of
// 1e-10 sigma_1 at the fp32 floor 2e-6 sigma_1 of the encoder.  A matrix with singular values at or under that floor
// (rank-deficient gradients), or with two kept atoms whose vectors are not separated (direct_vectors), is left to the
// Jacobi iteration: DS_ACCEPT stays 0.
#include <algorithm>
#include <array>
#include <cmath>
#include <vector>

#include "svd_device.h"
#include "svd_direct.h"

namespace atomo {
namespace direct {

using svd::Work;
using svd::floatx4;

namespace {

enum { CLS_64 = 0, CLS_128, CLS_256, CLS_512, CLS_640, CLS_COUNT };
// columns / 64, workgroups of the group
constexpr int CLS_CHUNKS[CLS_COUNT] = {1, 2, 4, 8, 10};
constexpr int XCH = 6;            // vectors in the exchange slots of a group, see Tri
constexpr int CLS_WGS[CLS_COUNT] = {1, 1, 16, 16, 32};
constexpr int HALFWAY = 384, FEW_WGS = 8;    // rows that groups of so many workgroups take up, in calls of many, see direct_tridiagonal_few
// of a vector in the exchange slots of a matrix: of its group, and of one of eight workgroups
__host__ __device__ inline int slot_entries(int cls)
{
    return 64 * CLS_CHUNKS[cls] + (cls <= CLS_128 ? 0 : cls == CLS_256 ? 256 : HALFWAY);
}

__device__ inline double fold8(double a, double b, int lane)
{
    const bool up = lane & 8;
    const double keep = up ? b : a, give = up ? a : b;
    return keep + dpp<DPP_ROR8>(give);
}
// K <= 8 sums over the 64 lanes at once: lane l receives sum number (l >> 5 & 1) | (l >> 4 & 1) << 1 | (l >> 3 & 1) << 2
template <int K>
__device__ inline double wave_sums(const double (&v)[K], int lane)
{
    constexpr int K1 = (K + 1) / 2, K2 = (K1 + 1) / 2;
    double a[K1], b[K2];
#pragma unroll
    for (int i = 0; i < K1; ++i) a[i] = fold32(v[2 * i], 2 * i + 1 < K ? v[2 * i + 1] : v[2 * i]);
#pragma unroll
    for (int i = 0; i < K2; ++i) b[i] = fold16(a[2 * i], 2 * i + 1 < K1 ? a[2 * i + 1] : a[2 * i]);
    return sum8(fold8(b[0], K2 > 1 ? b[1] : b[0], lane));
}
// K <= 64 sums over the 64 lanes at once: lane l receives sum number reverse6(l), in as many of its bits as K needs
// (there may be none of that number)
template <int K, typename Fold, typename Add>
__device__ inline void halve(const double (&in)[K], double (&out)[(K + 1) / 2], Fold fold, Add add)
{
#pragma unroll
    for (int i = 0; i < K / 2; ++i) out[i] = fold(in[2 * i], in[2 * i + 1]);
    if constexpr (K & 1) out[K / 2] = add(in[K - 1]);
}
template <int CTRL>
__device__ inline double fold_dpp(bool up, double a, double b)
{
    const double keep = up ? b : a, give = up ? a : b;
    return keep + dpp<CTRL>(give);
}
template <int K>
__device__ inline double lane_sums(const double (&v)[K], int lane)
{
    constexpr int K1 = (K + 1) / 2, K2 = (K1 + 1) / 2, K3 = (K2 + 1) / 2, K4 = (K3 + 1) / 2, K5 = (K4 + 1) / 2;
    static_assert(K5 <= 2, "a sum per lane");
    double a[K1], b[K2], c[K3], d[K4], e[K5], f[1];
    halve(v, a, [](double x, double y) { return fold32(x, y); }, [](double x) { return fold32(x, x); });
    halve(a, b, [](double x, double y) { return fold16(x, y); }, [](double x) { return fold16(x, x); });
    halve(b, c, [&](double x, double y) { return fold_dpp<DPP_ROR8>(lane & 8, x, y); }, [](double x) { return x + dpp<DPP_ROR8>(x); });
    halve(c, d, [&](double x, double y) { return fold_dpp<DPP_HALF_MIRROR>(lane & 4, x, y); }, [](double x) { return x + dpp<DPP_HALF_MIRROR>(x); });
    halve(d, e, [&](double x, double y) { return fold_dpp<DPP_XOR2>(lane & 2, x, y); }, [](double x) { return x + dpp<DPP_XOR2>(x); });
    halve(e, f, [&](double x, double y) { return fold_dpp<DPP_XOR1>(lane & 1, x, y); }, [](double x) { return x + dpp<DPP_XOR1>(x); });
    return f[0];
}
__host__ __device__ constexpr int reverse6(int l) { return (l & 1) << 5 | (l & 2) << 3 | (l & 4) << 1 | (l & 8) >> 1 | (l & 16) >> 3 | (l & 32) >> 5; }
__device__ inline int sum_slot(int lane) { return (lane >> 5 & 1) | (lane >> 4 & 1) << 1 | (lane >> 3 & 1) << 2; }

// ------------------------------------------------------------------------------------------------
// Gram matrix: partial sums of one 64 x 64 tile over one chunk of columns of A
// ------------------------------------------------------------------------------------------------
constexpr int GK = 32;           // columns staged per step
constexpr int GLD = GK + 4;      // row stride in LDS: 16 rows x 4 consecutive columns hit 64 different banks

// One row of A per lane group: loads the 64 x 32 piece (rows row0.., columns c0..) into registers / LDS.
// Rows before the padding and columns past c_end are zero.
struct GramLoader {
    Global<const float> G;
    long long ldg;
    int transposed, r;
    __device__ inline void fetch(float (&v)[8], int row0, int c0, int c_end, int tid) const
    {
        if (!transposed) {
            // thread: row tid / 4, eight columns from 8 (tid mod 4)
            const int row = row0 + (tid >> 2), c = c0 + 8 * (tid & 3);
            const Global<const float> g = G + (long long)row * ldg + c;
            if (row >= 0 && c + 8 <= c_end && ((((size_t)g) & 15) == 0)) {
                const floatx4 x = *(Global<const floatx4>)g, y = *(Global<const floatx4>)(g + 4);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    v[k] = x[k];
                    v[4 + k] = y[k];
                }
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = row >= 0 && c + k < c_end ? g[k] : 0.0f;
            }
        } else {
            // thread: row tid mod 64, columns tid / 64 + 4 k
            const int row = row0 + (tid & 63), c = c0 + (tid >> 6);
            const Global<const float> g = G + (long long)c * ldg + row;
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = row >= 0 && c + 4 * k < c_end ? g[(long long)(4 * k) * ldg] : 0.0f;
        }
    }
    __device__ inline void store(const float (&v)[8], float (*t)[GLD], int tid) const
    {
        if (!transposed) {
            float* p = &t[tid >> 2][8 * (tid & 3)];
            *(float4*)p = make_float4(v[0], v[1], v[2], v[3]);
            *(float4*)(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) t[tid & 63][(tid >> 6) + 4 * k] = v[k];
        }
    }
};

// What the kernels behind the Gram matrix need cleared; by the threads that finish its first tile.
__device__ inline void clear_for_steps(const DirectMat& m, int tid, int n_threads)
{
    const int N = m.nt * TILE;
    if (tid < DS_WORDS) m.st[tid] = 0;
    if (tid < 2) m.gate[tid] = 0;                                // (and the slots of both groups)
    for (int i = tid; i < XCH * slot_entries(m.cls); i += n_threads) m.xch[i] = 0;
    if (tid < m.pad) m.td[tid] = make_double2(0.0, 2.0);
    if (tid == m.pad) m.td[tid].x = 0.0;
    // rows of the reflectors' blocks that are no step
    for (int i = tid; i < (m.pad & 15) * N; i += n_threads) m.refl[(size_t)(m.pad & ~15) * N + i] = 0.0;
    for (int i = tid; i < 2 * N; i += n_threads) m.refl[(size_t)(N - 2) * N + i] = 0.0;
}

// Bound: the double-precision matrix cores (2 x 64 cycles of v_mfma_f64_16x16x4 per 16 columns, sub-tile and wave; the
// operand of four instructions is one 16-byte LDS read per lane).  A wave owns a 32 x 32 quarter of the tile.
__global__ __launch_bounds__(256) void direct_gram(const DirectMat* mats, const Work* work)
{
    __shared__ float ta[64][GLD], tb[64][GLD];
    const Work wk = work[blockIdx.x];
    const DirectMat& m = mats[wk.mat];
    const int ti = wk.a, tj = wk.b, chunk = wk.c;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, q = lane >> 4;
    const int qi = (wave >> 1) * 32, qj = (wave & 1) * 32;
    const GramLoader ld{global(m.G), m.ldg, m.transposed, m.r};
    const int rowa = ti * TILE - m.pad, rowb = tj * TILE - m.pad;
    const int c0 = chunk * m.kchunk, c1 = min(m.M, c0 + m.kchunk);
    const bool same = ti == tj;
    doublex4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
    float va[8], vb[8];
    ld.fetch(va, rowa, c0, c1, tid);
    if (!same) ld.fetch(vb, rowb, c0, c1, tid);
    for (int c = c0; c < c1; c += GK) {
        __syncthreads();
        ld.store(va, ta, tid);
        if (!same) ld.store(vb, tb, tid);
        __syncthreads();
        if (c + GK < c1) {
            ld.fetch(va, rowa, c + GK, c1, tid);
            if (!same) ld.fetch(vb, rowb, c + GK, c1, tid);
        }
        float (*tbb)[GLD] = same ? ta : tb;
#pragma unroll
        for (int h = 0; h < GK / 16; ++h) {
            float4 a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = *(const float4*)&ta[qi + 16 * i + l16][16 * h + 4 * q];
                b[i] = *(const float4*)&tbb[qj + 16 * i + l16][16 * h + 4 * q];
            }
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const float ax = x == 0 ? a[i].x : x == 1 ? a[i].y : x == 2 ? a[i].z : a[i].w;
                        const float bx = x == 0 ? b[j].x : x == 1 ? b[j].y : x == 2 ? b[j].z : b[j].w;
                        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)ax, (double)bx, acc[i][j], 0, 0, 0);
                    }
        }
    }
    const int ntiles = m.nt * (m.nt + 1) / 2, tile = ti * m.nt - ti * (ti - 1) / 2 + (tj - ti);
    const Global<double> out = global(m.part) + ((size_t)chunk * ntiles + tile) * (TILE * TILE);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) out[(qi + 16 * i + 4 * v + q) * TILE + qj + 16 * j + l16] = acc[i][j][v];
}

// Adds the partial tiles up in the order of the columns and writes both triangles; a workgroup takes 16 rows of a tile.
// Bound: HBM read where there are many tiles (the ResNet-18 layers 16 -> 14 us, 601 x 1237 and smaller ones 13.4 -> 7.9 against a
// workgroup per tile and one partial tile at a time); with one tile the round trips for the partial sums, five at a time: 4.3 us
// for the nine of 64 x 576 (7.5 by one workgroup).
constexpr int SUM_ROWS = 16, SUM_AHEAD = 5;
__global__ __launch_bounds__(256) void direct_gram_sum(const DirectMat* mats, const Work* work)
{
    __shared__ double t[SUM_ROWS][TILE + 1];
    const Work wk = work[blockIdx.x];
    const DirectMat& m = mats[wk.mat];
    const int ti = wk.a, tj = wk.b, row0 = SUM_ROWS * wk.c, tid = threadIdx.x, N = m.nt * TILE;
    constexpr int PER = SUM_ROWS * TILE / 256;
    const int ntiles = m.nt * (m.nt + 1) / 2, tile = ti * m.nt - ti * (ti - 1) / 2 + (tj - ti);
    const Global<const double> in = global((const double*)m.part) + (size_t)tile * (TILE * TILE) + row0 * TILE + tid;
    const Global<double> C = global(m.C);
    const size_t stride = (size_t)ntiles * (TILE * TILE);
    double sum[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) sum[p] = 0.0;
    for (int c = 0; c < m.nchunks; c += SUM_AHEAD) {
        double x[SUM_AHEAD][PER];
#pragma unroll
        for (int u = 0; u < SUM_AHEAD; ++u)
#pragma unroll
            for (int p = 0; p < PER; ++p) x[u][p] = in[(size_t)min(c + u, m.nchunks - 1) * stride + 256 * p];
#pragma unroll
        for (int u = 0; u < SUM_AHEAD; ++u)
#pragma unroll
            for (int p = 0; p < PER; ++p) sum[p] += c + u < m.nchunks ? x[u][p] : 0.0;
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int i = (tid >> 6) + 4 * p, j = tid & 63;
        C[(size_t)(ti * TILE + row0 + i) * N + tj * TILE + j] = sum[p];
        t[i][j] = sum[p];
    }
    __syncthreads();
    if (ti == tj) {
        if (tid < SUM_ROWS) m.diag[ti * TILE + row0 + tid] = t[tid][row0 + tid];
    } else {
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int i = tid / SUM_ROWS + 256 / SUM_ROWS * p, j = tid % SUM_ROWS;
            C[(size_t)(tj * TILE + i) * N + ti * TILE + row0 + j] = t[j][i];
        }
    }
    if (ti == 0 && tj == 0) clear_for_steps(m, tid + 256 * wk.c, 256 * (TILE / SUM_ROWS));
}

// A partial tile is on its way to whoever adds them up, on any die: stores and loads of agent scope.
__device__ inline void put_part(Global<double> p, double x)
{
    __hip_atomic_store((Global<u64>)p, (u64)__double_as_longlong(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline double get_part(Global<const double> p)
{
    return __longlong_as_double((long long)__hip_atomic_load((Global<const u64>)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
// True for the last of a tile's chunks to be finished, in the one thread that asks, between wait_for_stores and loads_from_here.
__device__ inline bool last_chunk(const DirectMat& m, int tile)
{
    return __hip_atomic_fetch_add(global(m.tickets) + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)m.nchunks - 1u;
}
// What the wave has put is where every die's loads of agent scope look, before anything that follows (vmcnt(0), the other counters
// as they are: a relaxed store of agent scope that is acknowledged is there).  The fences cost no instruction: the compiler moves
// neither the stores past the wait nor the wait's successors, nor loads, in front of it.
__device__ inline void wait_for_stores()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
__device__ inline void loads_from_here() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront"); }

// The same sums, bit for bit, for calls of many tiles: a tile per wave, the data straight from the caches into registers, no barrier.
// Bound: the matrix cores again, in whose 64 cycles the vector unit of the same SIMD does nothing: every other instruction comes on
// top (measured: 66 cycles alone, 73 with one conversion from float beside it, 80 with two).  direct_gram has one conversion per
// matrix instruction and more around it, this one 40 instructions per 64 of them, and leaves out the sub-tiles below the diagonal.
// The last wave of a tile adds the partial tiles up beside the matrix instructions of the other wave on its SIMD.
// 64 x (512 x 4608), calls one after the other: 1331 us, of direct_gram and direct_gram_sum 1400 + 140; without the sums, which
// direct_gram_sum then takes 138 us for, 1233.  Wide matrices (rows of A contiguous) whose chunks are whole 16s of columns.  A wave takes a tile of a chunk
// of 576 columns 63 us or, two on a SIMD, twice that, so the call has to have many (WIDE_MIN); and the partial tiles that go through
// memory, 32 KB each way, cost as much for a chunk of few columns as for one of many (WIDE_COLUMNS).
// (The same hand-over in place of direct_gram_sum behind direct_gram: 64 x 576 14.4 -> 16.9 us, the ResNet-18 layers 124 -> 139:
// stores of agent scope write through.)
typedef float floatx4_any __attribute__((ext_vector_type(4), aligned(4)));
template <bool SAME>
__device__ inline void wide_tile(const DirectMat& m, int ti, int tj, int chunk, int lane)
{
    const int ntiles = m.nt * (m.nt + 1) / 2, tile = ti * m.nt - ti * (ti - 1) / 2 + (tj - ti);
    const size_t chunk_size = (size_t)ntiles * (TILE * TILE);
    const Global<double> part = global(m.part) + (size_t)tile * (TILE * TILE);
    const long long ld = m.ldg;
    const int c0 = chunk * m.kchunk, cols = min(m.M - c0, m.kchunk);
    const Global<const float> A = global(m.G) + (long long)(ti * TILE - m.pad) * ld + c0;
    const Global<const float> B = global(m.G) + (long long)(tj * TILE - m.pad) * ld + c0;
    const int l16 = lane & 15, q = lane >> 4;
    const unsigned offset = 4u * ((unsigned)l16 * (unsigned)ld + 4u * q);
    doublex4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
    floatx4 a[4], b[4];
    // lane (l16, q): columns c + 4 q .. c + 4 q + 3 of rows 16 i + l16
    auto fetch = [&](int c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = *(Global<const floatx4_any>)((Global<const char>)(A + 16 * i * ld + c) + offset);
            if (!SAME) b[i] = *(Global<const floatx4_any>)((Global<const char>)(B + 16 * i * ld + c) + offset);
        }
    };
    fetch(0);
    for (int c = 0; c < cols; c += 16) {
        double da[4][4], db[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                da[i][x] = (double)a[i][x];
                db[i][x] = SAME ? da[i][x] : (double)b[i][x];
            }
        __builtin_amdgcn_sched_barrier(0);
        fetch(min(c + 16, cols - 16));
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = SAME ? i : 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(da[i][x], db[j][x], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = SAME ? i : 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) put_part(part + chunk * chunk_size + (16 * i + 4 * v + q) * TILE + 16 * j + l16, acc[i][j][v]);
    wait_for_stores();
    int last = 0;
    if (lane == 0) last = last_chunk(m, tile);
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    loads_from_here();
    // (all loads of a partial tile in flight at once, beside the matrix instructions of the other wave)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = SAME ? i : 0; j < 4; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
    for (int c = 0; c < m.nchunks; ++c) {
        doublex4 t[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = SAME ? i : 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) t[i][j][v] = get_part((Global<const double>)part + c * chunk_size + (16 * i + 4 * v + q) * TILE + 16 * j + l16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = SAME ? i : 0; j < 4; ++j) acc[i][j] += t[i][j];
    }
    const int N = m.nt * TILE;
    const Global<double> C = global(m.C);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = SAME ? i : 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * i + 4 * v + q, col = 16 * j + l16;
                C[(size_t)(ti * TILE + row) * N + tj * TILE + col] = acc[i][j][v];
                if (!SAME || i != j) C[(size_t)(tj * TILE + col) * N + ti * TILE + row] = acc[i][j][v];
                if (SAME && i == j && row == col) m.diag[ti * TILE + row] = acc[i][j][v];
            }
    if (SAME && ti == 0) clear_for_steps(m, lane, 64);
}

// In front of direct_gram_wide, a workgroup per matrix: its tickets in the workspace are what earlier calls left there.
__global__ __launch_bounds__(64) void direct_clear_tickets(const DirectMat* mats)
{
    const DirectMat& m = mats[blockIdx.x];
    for (int i = threadIdx.x; i < m.nt * (m.nt + 1) / 2; i += 64) m.tickets[i] = 0;
}

__global__ __launch_bounds__(256, 2) void direct_gram_wide(const DirectMat* mats, const Work* work, int n)
{
    const int item = 4 * blockIdx.x + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (item >= n) return;
    const Work wk = work[item];
    if (wk.mat < 0) return;
    const DirectMat& m = mats[wk.mat];
    const int lane = threadIdx.x & 63;
    if (wk.a == wk.b) wide_tile<true>(m, wk.a, wk.b, wk.c, lane);
    else wide_tile<false>(m, wk.a, wk.b, wk.c, lane);
}

// ------------------------------------------------------------------------------------------------
// Householder reduction C = H T H^T
// ------------------------------------------------------------------------------------------------
// Where the steps are kept.
struct StepStore {
    Global<double> refl, tau, td, od;
    int N;
    __device__ inline StepStore(const DirectMat& m)
        : refl(global(m.refl)), tau(global(m.tau)), td(global((double*)m.td)), od(global(m.od)), N(m.nt * TILE) {}
    // entry k of the tridiagonal matrix and its coupling to entry k + 1
    __device__ inline void put(int k, double t, double d, double beta) const
    {
        tau[k] = t;
        td[2 * k + 1] = d;
        od[k] = beta;
        td[2 * k + 2] = fmax(beta * beta, OD2_MIN);
    }
};

// What every wave works out for itself before the first step: the scale of the matrix (a power of four that brings the
// trace under 1) and how many of its rows are zero.
template <int C>
__device__ inline double scale_of(const DirectMat& m, int off, int lane, int& expo, int& zero_rows)
{
    const int N = m.nt * TILE;
    double tr = 0.0;
    int zeros = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int i = lane + 64 * c - off;
        const double d = i >= 0 ? global(m.C)[(size_t)i * N + i] : 0.0;
        tr += d;
        zeros += __popcll(__ballot(i >= m.pad && d == 0.0));
    }
    tr = wave_sum(tr);
    int e = 0;
    if (tr > 0.0 && tr <= 1.7976931348623157e308) (void)frexp(tr, &e);
    e += e & 1;
    expo = e;
    zero_rows = zeros;
    return ldexp(1.0, -e);
}

// Groups of 8, 16 or 32 workgroups (matrices of more than 128 rows, until 64 are left): every wave owns R rows of the matrix in
// registers (lane l: columns l, l + 64, ..), row r belonging to wave r mod W, and works the whole vectors x, v, w out for itself, all
// waves the same bits; one exchange per step: every wave publishes the entries of A y of its rows (y: the column below its first entry;
// A v = A y + v0 A e_{k+1}, so the reflector need not be known), the owner of row k + 1 that row, and every workgroup reads all of
// both, a quarter per wave.
// What everybody waits for is (A y)_i, so a step does nothing else before it: the product is taken with the matrix as it was before the
// last step's update, whose share is a product with two sums of y (v_i (w y) + w_i (v y)).  The update itself, the reflector and the
// row of the next step (handed over a step early, the readers add the update that it lacks) come behind it, while the entries
// travel; the loads that look for them go out in the middle of that work (a load of 512 bytes by every wave takes 250 cycles, four of
// them 460, whether the entries are there or not; a look that is too early costs a second one, at the entries of A y alone: the row has
// been there for a step; one step in three has one).  The ResNet-18 layers, the figures of a sentence from one card each.  With the look there
// 468 us, behind the reflector's vector 495, in front of the update 575, two looks on their way at once 485.  With the second look at the
// entries alone 452, at the row too 467 (601 x 1237 and smaller ones 594 and 609).
// An entry is one 8-byte store whose two lowest mantissa bits carry a tag that tells it from the one that lay there before: a reader
// knows from the value that it is the one of this step, no flag and no second round trip.  Two slots for A y by step parity: a wave
// that publishes step k + 1 has read all of step k, so when a wave has read all of step k + 1 nobody needs slot k any more; four for
// the rows, which are written a step ahead.
// The workgroups of a group sit on one die (blockIdx mod 8), whose L2 the exchange goes through: 0.77 us per step among 64
// waves, against 5 us through memory; they check that with the die's number, and store through to memory if it is not so.
// (On one die the stores have workgroup scope, which the memory model does not extend to other workgroups.  What carries them
// over is the hardware: vector stores write through the L1 to the L2 that the whole die shares, and the readers' loads, of
// agent scope, do not hit in an L1.  Agent scope on the stores would send them through to memory as well.)
// Waits: nothing guarantees that a group is resident as a whole - other work on the GPU can hold the places that its last
// workgroups need, and partial groups of three calls can hold each other's.  So every wait has a bound, and a group that does
// not come together leaves as one (Gate); the last of its workgroups to start reduces the matrix alone.
// Bound: what a wave does for itself in a step, one wave on every SIMD: without the waits for the others a step takes as long.  448
// steps of 512 rows on 128 waves: 3000 cycles each at the beginning and 2000 at the end, 442 us in all in the profile of the ResNet-18 step.
// What it was before, each pair from one card: 452 instead of 446 with the loop where the compiler puts it; 517 instead of 468 with a chain of
// branches and v_readlane for what a vector holds at the wave's rows, a reduction of its own for the norm, and the reflector in front of the
// update (800 of 3500 cycles).  Rows and columns split between the
// waves of a workgroup, two instead of eight entries of a vector per lane: 566, for a second barrier and sums of sixteen rows.  Four
// groups per die, two waves on every SIMD: the issue of the vectors that every wave works out for itself (direct_tridiagonal_few).
//
// The word that a group starts by: seven bits per die count the workgroups that have started on it; OFF, set by one that has
// waited too long, holds for all of them: it is only set while some are missing, and who finds it set does not go on.  The
// last to start then knows that no other has done or will do anything.
struct Gate {
    static constexpr u64 OFF = 1ull << 63;
    static __device__ inline int on_die(u64 word, int die) { return (int)(word >> (7 * die)) & 127; }
    static __device__ inline int started(u64 word)
    {
        int sum = 0;
#pragma unroll
        for (int d = 0; d < 8; ++d) sum += on_die(word, d);
        return sum;
    }
    static __device__ inline int this_die() { return (int)__builtin_amdgcn_s_getreg(20 | (31 << 11)) & 7; }
    // True in thread 0 of the last workgroup to start, if the group does not go on.  (No time to wait at all, ticks == 0: the
    // group gives up however fast it is.)
    static __device__ inline bool start(Global<u64> gate, int n_wgs, long long ticks)
    {
        if (threadIdx.x != 0) return false;
        if (ticks == 0) __hip_atomic_fetch_or(gate, OFF, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const u64 before = __hip_atomic_fetch_add(gate, 1ull << (7 * this_die()), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return (before & OFF) && started(before) == n_wgs - 1;
    }
    // True once all have started (one_die: all of them on this workgroup's die), false if the group does not go on.
    static __device__ inline bool pass(Global<u64> gate, int n_wgs, long long ticks, bool& one_die)
    {
        const int die = this_die();
        const long long t0 = wall_clock64();
        while (true) {
            u64 word = __hip_atomic_load(gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (word & OFF) return false;
            if (started(word) == n_wgs) {
                one_die = on_die(word, die) == n_wgs;
                return true;
            }
            if (wall_clock64() - t0 >= ticks)                    // (a word that has changed meanwhile is looked at again)
                (void)__hip_atomic_compare_exchange_strong(gate, &word, word | OFF, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_s_sleep(4);
        }
    }
};

constexpr int TAIL = 64;                                         // rows that a group leaves
constexpr int ONE = 128, TS = ONE / 16;                          // rows of TriOne; slots of 16

// How a workgroup's part in a reduction ends: done; a wait of a step gave up; the group did not go on, and this workgroup was
// the last of it to start, or not.
enum TriEnd { TRI_DONE, TRI_FAILED, TRI_LAST, TRI_LEFT };

// A group of W waves for the last 64 C rows, until LEFT are left.  One of eight workgroups (FEW) may go on from what another has left:
// the matrix without the last step's update, and the vectors that it needs for that, so that the sums stay the same.  Every matrix has
// the same bits whatever the number of workgroups: a sum over a row is one wave's, in the order of the columns.
template <int C, int R, int W, int LEFT = TAIL>
struct Tri {
    static constexpr int CN = 64 * C, OWN = (C + 3) / 4;
    static constexpr int LAST = C - LEFT / 64 - 1;               // the last chunk of columns that is reduced here
    static constexpr int TURN = W < 64 ? W : 64;                 // rows that the waves hand over in turn
    static constexpr bool FEW = W == 4 * FEW_WGS;
    static_assert(W * R == CN, "every row has a wave");
    // Measured, and not explained by the number of instructions where a wave has few rows: ResNet-18, four rows, 458 us with KEEP and 476
    // without (the same look); 64 x (512 x 4608), eight and twelve rows, bound by issue, 639 + 627 and 617 + 602.
    static constexpr bool KEEP = R <= 5;
    double a[R][C];
    // Column k; the last step's vectors, which the rows have still to be updated with.  [C]: their entries at the wave's rows, row
    // slot t in lane t of every row of 16 lanes, from where they are broadcast.
    double x[C + 1], v[C + 1], wv[C + 1];
    double tau, diagonal, beta;      // the last step's
    Global<u64> slots;
    double2 (*shared)[CN];           // [2][CN] by step parity: p and column k + 1
    int lane, wave, member, w, off, k_first, spin_limit;
    int row_turn, keep_turn;         // the next steps at which this wave hands over a row, its workgroup keeps a vector
    int row_number;                  // the row of this lane in the vectors' last part
    bool local;                      // the group sits on one die

    static __device__ inline u64 entry(double value, u64 tag) { return ((u64)__double_as_longlong(value) & ~3ull) | tag; }
    static __device__ inline double value(u64 entry) { return __longlong_as_double((long long)(entry & ~3ull)); }
    static __device__ inline Global<u64> at_byte(Global<u64> slot, unsigned byte) { return (Global<u64>)((Global<char>)slot + byte); }
    __device__ inline void put(Global<u64> p, u64 entry) const
    {
        __hip_atomic_store(p, entry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__builtin_expect(!local, 0)) __hip_atomic_store(p, entry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // a row of the matrix, in row slot T of this wave
    template <int P, int T>
    __device__ inline void put_row(Global<u64> slot, u64 tag) const
    {
#pragma unroll
        for (int c = P; c < C; ++c) put(slot + lane + 64 * c, entry(a[T][c], tag));
    }
    // row `row` = k + 2 of this wave, k a step of phase P
    template <int P, int T = 64 * P / W>
    __device__ __forceinline__ void put_turn(int row, Global<u64> slot, u64 tag) const
    {
        if constexpr (W >= 64) {
            constexpr int Q = W / 64;
            if (row < 64 * (P + 1)) {
                if (w >> 6 == P % Q) put_row<P, P / Q>(slot, tag);
            } else if (w >> 6 == (P + 1) % Q) {
                put_row<P, (P + 1) / Q>(slot, tag);
            }
        } else if constexpr (T <= 64 * (P + 1) / W && T < R) {   // (up to the first row of chunk P + 1)
            if (w + W * T == row) put_row<P, T>(slot, tag);
            else put_turn<P, T + 1>(row, slot, tag);
        }
    }
    template <int T>
    __device__ inline void put_first(int row) const
    {
        if (w + W * T == row) put_row<0, T>(slot_c(1), 1);
        if constexpr (T + 1 < R) put_first<T + 1>(row);
    }
    // where the entries of A y and of the column of a step lie, and their tags (a cleared slot has tag 0; steps count from 1)
    __device__ inline Global<u64> slot_p(unsigned step) const { return slots + (step & 1) * CN; }
    __device__ inline Global<u64> slot_c(unsigned step) const { return slots + (2 + (step & 3)) * CN; }
    static __device__ inline unsigned tag_p(unsigned step) { return step & 3; }
    static __device__ inline unsigned tag_c(unsigned step) { return (step >> 2) + 1 & 3; }
    // f(integral_constant T) for the row slots from T0 on
    template <int T0, typename F>
    static __device__ __forceinline__ void for_slots(F&& f)
    {
        if constexpr (T0 < R) {
            f(std::integral_constant<int, T0>());
            for_slots<T0 + 1>(f);
        }
    }
    // The entries of A y at the wave's rows, and the update.  KEEP: what the last step's vectors are at those rows stays in registers from the
    // one to the other.  Else it is broadcast inside the products; one right behind the product that it adds to would wait for that, and the
    // compiler does not know: the two of an entry stand apart.
    template <int P, int T0, int K>
    __device__ __forceinline__ void products(const double (&y)[C + 1], double vy, double wy, double (&sum)[K], double (&wr)[R], double (&vr)[R]) const
    {
        for_slots<T0>([&](auto t) {
            constexpr int T = decltype(t)::value;
            double s = a[T][P] * y[P];
#pragma unroll
            for (int c = P + 1; c < C; ++c) s = fma(a[T][c], y[c], s);
            if constexpr (KEEP) {
                wr[T] = row_lane<T>(wv[C]);
                vr[T] = row_lane<T>(v[C]);
                s = fma(-wr[T], vy, fma(-vr[T], wy, s));
            }
            sum[T - T0] = s;
        });
        if constexpr (!KEEP) {
            for_slots<T0>([&](auto t) { sub_lane_product<decltype(t)::value>(sum[t - T0], v[C], wy); });
            for_slots<T0>([&](auto t) { sub_lane_product<decltype(t)::value>(sum[t - T0], wv[C], vy); });
        }
    }
    template <int P, int T0>
    __device__ __forceinline__ void update(const double (&wr)[R], const double (&vr)[R])
    {
        for_slots<T0>([&](auto t) {
            constexpr int T = decltype(t)::value;
            if constexpr (KEEP) {
#pragma unroll
                for (int c = P; c < C; ++c) {
                    a[T][c] = fma(-wr[T], v[c], fma(-vr[T], wv[c], a[T][c]));
                    here(a[T][c]);
                }
            } else {
#pragma unroll
                for (int c = P; c < C; ++c) sub_lane_product<T>(a[T][c], v[C], wv[c]);
#pragma unroll
                for (int c = P; c < C; ++c) {
                    sub_lane_product<T>(a[T][c], wv[C], v[c]);
                    here(a[T][c]);
                }
            }
        });
    }

    // step k - 1, every wave of the workgroup a part; with zeros in what is finished of its vector (that is read in pairs of chunks)
    template <int P>
    __device__ __forceinline__ void keep(int k, const StepStore& store) const
    {
        const int kk = k - 1 - off;
        const Global<double> row = store.refl + (size_t)kk * store.N - off + lane;
#pragma unroll
        for (int c = P > 1 ? P - 2 : 0; c < C; ++c)
            if ((c & 3) == wave && (c >= P || 64 * c >= off)) row[64u * c] = c < P ? 0.0 : v[c < P ? P : c];
        if constexpr (FEW && P <= 1) {                           // (the chunk in front, another group's)
            if (off < 0 && wave == 3) *(row - 64) = 0.0;
        }
        if (wave == 3 && lane == 0) store.put(kk, tau, diagonal, beta);
    }

    // steps k of [64 P, 64 (P + 1)): chunks of columns before P are finished
    template <int P>
    __device__ __forceinline__ void phase(int& k, const StepStore& store)
    {
        constexpr int T0 = 64 * P / W;                           // row slots before T0 are finished
        constexpr int PN = P + 1;
        constexpr int K = R - T0 + 1;                            // sums of a step: the entries of A y, and y y
        constexpr int J0 = P / 4, L = OWN - J0;
        // this wave's chunks of p and of the column (one of a finished chunk: any other)
        unsigned at[L];
#pragma unroll
        for (int j = 0; j < L; ++j) at[j] = 8u * (unsigned)(lane + 64 * min(max(wave + 4 * (j + J0), P), C - 1));
        const int row_at = max(row_number, 64 * P);
        // (a sum is in several lanes, the first of them hands it over)
        const unsigned sum_at = 8u * (unsigned)(w + W * (T0 + reverse6(lane)));
        const bool mine = reverse6(lane) < R - T0;
        for (; k < 64 * PN; ++k) {
            const int k1 = k + 1;
            const bool next_chunk = k1 == 64 * PN;               // row k + 1 is the first of chunk P + 1
            const unsigned step = (unsigned)(k - k_first + 1);
            u64 pu[L], cu[L];
            auto look_p = [&]() {
#pragma unroll
                for (int j = 0; j < L; ++j) pu[j] = __hip_atomic_load(at_byte(slot_p(step), at[j]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            auto look_c = [&]() {
#pragma unroll
                for (int j = 0; j < L; ++j) cu[j] = __hip_atomic_load(at_byte(slot_c(step), at[j]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            double y[C + 1], sum[K], wr[R], vr[R], vy = 0.0, wy = 0.0, sq = 0.0;
            if constexpr (!KEEP) broadcasts(v[C], wv[C]);
#pragma unroll
            for (int c = P; c < C; ++c) {
                y[c] = c > PN || lane + 64 * c > k1 ? x[c] : 0.0;
                vy = fma(v[c], y[c], vy);
                wy = fma(wv[c], y[c], wy);
                sq = fma(y[c], y[c], sq);
            }
            products<P, T0>(y, vy, wy, sum, wr, vr);
            sum[K - 1] = sq;
            const double sums = lane_sums<K>(sum, lane);
            if (mine) put(at_byte(slot_p(step), sum_at), entry(sums, tag_p(step)));
            // behind what the others wait for: the last step's vector (one workgroup keeps it for the way back), the reflector beside
            // the matrix, the row that the next step hands over
            __builtin_amdgcn_sched_barrier(0);
            look_c();
            if (__builtin_expect(k == keep_turn, 0)) {
                keep<P>(k, store);
                keep_turn += W / 4;
            }
            const double sig2 = lane_value(sums, reverse6(K - 1)), alpha = lane_value(next_chunk ? x[PN] : x[P], k1 & 63);
            double v0;
            householder(alpha, sig2, beta, v0);
            tau = householder_tau(sig2, v0);
            update<P, T0>(wr, vr);
            here(v0);
            here(tau);
            if (__builtin_expect(k == row_turn, 0)) {
                put_turn<P>(k + 2, slot_c(step + 1), tag_c(step + 1));
                row_turn += TURN;
            }
            __builtin_amdgcn_sched_barrier(0);
            look_p();
            __builtin_amdgcn_sched_barrier(0);
            diagonal = lane_value(x[P], k & 63);
            double fresh[C + 1];                                 // what the row of this step lacks of the last step's update
            {
                const double v1 = lane_value(next_chunk ? v[PN] : v[P], k1 & 63), w1 = lane_value(next_chunk ? wv[PN] : wv[P], k1 & 63);
#pragma unroll
                for (int c = P; c <= C; ++c) {
                    fresh[c] = fma(-w1, v[c], -v1 * wv[c]);
                    here(fresh[c]);
                }
            }
            y[C] = row_number > k1 ? x[C] : 0.0;
#pragma unroll
            for (int c = P; c <= C; ++c) {
                v[c] = c == C ? (row_number == k1 ? v0 : y[c]) : c <= PN && lane + 64 * c == k1 ? v0 : y[c];
                here(v[c]);
            }
            __builtin_amdgcn_sched_barrier(0);
            auto ready = [&]() {
                unsigned other = 0;
#pragma unroll
                for (int j = 0; j < L; ++j) other |= ((unsigned)pu[j] ^ tag_p(step)) | ((unsigned)cu[j] ^ tag_c(step));
                return __all((other & 3u) == 0u);
            };
            if (__builtin_expect(!ready(), 0)) {
                look_p();                                        // (the row of this step is there already, as a rule)
                for (int spins = 0; !ready(); look_p(), look_c())
                    if (++spins > spin_limit) {                  // (once: the steps after it wait for nothing)
                        spin_limit = 0;
                        break;
                    }
            }
            double2* sh = shared[step & 1];
#pragma unroll
            for (int j = 0; j < L; ++j) sh[at[j] / 8] = make_double2(value(pu[j]), value(cu[j]));
            __syncthreads();
            double2 pc[C + 1];
#pragma unroll
            for (int c = P; c <= C; ++c) pc[c] = sh[c < C ? lane + 64 * c : row_at];
            __builtin_amdgcn_sched_barrier(0);                   // (all of them are on their way at once)
            double p[C + 1], gamma = 0.0;
#pragma unroll
            for (int c = P; c <= C; ++c) {
                x[c] = pc[c].y + fresh[c];
                p[c] = fma(v0, x[c], pc[c].x);
                if (c == C) p[c] = row_number <= k ? 0.0 : p[c];
                else if (c <= PN) p[c] = lane + 64 * c <= k ? 0.0 : p[c];
                if (c < C) gamma = fma(v[c], p[c], gamma);
            }
            const double pk1 = tau * lane_value(next_chunk ? p[PN] : p[P], k1 & 63);
            gamma = wave_sum(gamma) * (tau * (0.5 * tau));
            const double wk1 = fma(-gamma, v0, pk1);
#pragma unroll
            for (int c = P; c <= C; ++c) {
                wv[c] = fma(-gamma, v[c], tau * p[c]);
                x[c] = fma(-wv[c], v0, fma(-v[c], wk1, x[c]));
            }
        }
    }

    template <int P>
    __device__ __forceinline__ void phases(int& k, const StepStore& store)
    {
        phase<P>(k, store);
        if constexpr (P < LAST) phases<P + 1>(k, store);
    }

    static constexpr int SPIN_STEP = 1 << 20;                    // a quarter of a second and more: never seen

    __device__ __forceinline__ TriEnd run(const DirectMat& mm, int number, int n_wgs, long long start_ticks, double2* lds)
    {
        member = number;
        const StepStore store(mm);
        const int N = store.N;
        spin_limit = SPIN_STEP;
        shared = (double2(*)[CN])lds;
        lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        w = member * 4 + wave;
        row_number = w + W * min(lane & 15, R - 1);
        off = CN - N;
        slots = global(mm.xch) + (FEW ? XCH * 64 * CLS_CHUNKS[mm.cls] : 0);
        const bool last = Gate::start(global(mm.gate) + FEW, n_wgs, start_ticks);
        int expo = 0, zeros = 0;
        double scale = 1.0;                                      // (what another group has left is scaled)
        if (!FEW || off >= 0) scale = scale_of<C>(mm, off, lane, expo, zeros);
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const int i = w + W * t - off;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int j = lane + 64 * c - off;
                a[t][c] = i >= 0 && j >= 0 ? scale * global(mm.C)[(size_t)i * N + j] : 0.0;
            }
        }
        int k = !FEW || off >= 0 ? off + mm.pad : 0;
        k_first = k;
        // (a wave has its rows of a chunk once, its workgroup every (W / 4)th vector from the first step's on)
        row_turn = k + (w - (k + 2) & (TURN - 1));
        keep_turn = k + 1 + (member - k & (W / 4 - 1));
        const bool goes_on = FEW && off < 0;
        const Global<const double> column = goes_on ? global((const double*)mm.half) : global((const double*)mm.C) + (size_t)mm.pad * N - off;
        const Global<const double> last_v = goes_on ? column + CN : global((const double*)mm.C) + CN;
#pragma unroll
        for (int c = 0; c <= C; ++c) {
            const int i = c < C ? lane + 64 * c : row_number;
            x[c] = i >= off ? scale * column[i] : 0.0;
            v[c] = goes_on ? last_v[i] : 0.0;
            wv[c] = goes_on ? last_v[CN + i] : 0.0;
        }
        if (!Gate::pass(global(mm.gate) + FEW, n_wgs, start_ticks, local)) return __syncthreads_or(last) ? TRI_LAST : TRI_LEFT;
        put_first<0>(k + 1);
        phases<0>(k, store);
        // what is left goes back to memory
        constexpr int T0 = 64 * (LAST + 1) / W;
        if (k == keep_turn) keep<LAST + 1>(k, store);
        if constexpr (LEFT == TAIL) {
            double wr[R], vr[R];
            if constexpr (!KEEP) broadcasts(v[C], wv[C]);
            else for_slots<T0>([&](auto t) { wr[t] = row_lane<decltype(t)::value>(wv[C]), vr[t] = row_lane<decltype(t)::value>(v[C]); });
            update<LAST + 1, T0>(wr, vr);
        } else if (w == 0) {
#pragma unroll
            for (int c = LAST + 1; c < C; ++c) {
                const Global<double> at = global(mm.half) + lane + 64 * (c - LAST - 1);
                at[0] = x[c];
                at[LEFT] = v[c];
                at[2 * LEFT] = wv[c];
            }
        }
#pragma unroll
        for (int t = T0; t < R; ++t) {
            const Global<double> row = global(mm.C) + (size_t)(w + W * t - off) * N + lane - off;
            if (W * t + w >= CN - LEFT) {
#pragma unroll
                for (int c = LAST + 1; c < C; ++c) row[64 * c] = a[t][c];
            }
        }
        if ((!FEW || off >= 0) && w == 0 && lane == 0) {
            mm.st[DS_EXP] = expo;
            mm.st[DS_ZERO_ROWS] = zeros;
        }
        return spin_limit != 0 ? TRI_DONE : TRI_FAILED;
    }
};

// Up to 128 rows, or what a group leaves of a larger matrix: one workgroup of 256 threads, no exchange through memory.
// A thread holds rows 16 a + 4 wave + lane / 16 and columns 16 b + column_of(lane) of the trailing matrix, a, b < 8: the
// columns are dealt to the lanes of a row of 16 such that the first lane has the one with the number of the thread's own
// row, so what a vector holds at a row is a broadcast inside the row of lanes (row_newbcast) of what it holds at a column.  Every
// thread works the vectors out at its columns for itself, all with the same bits: sums over the sixteen lanes go through
// rotations, which give the same sum whatever column a row of lanes begins with.
// One barrier per step.  What is handed over is (A y)_i, y the column below its first entry, and column k + 1 before the
// step: the reflector v = y + v0 e_{k+1} is wanted only behind the barrier (A v = A y + v0 A e_{k+1}), so that the norm, the root
// and the reciprocal run beside the products.
// All waves do the same in a step, but for the three numbers that one of them keeps: the column is handed over by the lanes that have
// it, one of every row, and every row of lanes keeps the vector's entries at its rows.
// Bound: a step of 64 rows is a chain of about 250 instructions with one wave on every SIMD, 0.53 us; at 128 rows it is the issue of
// 500, 192 of them the fma of the matrix, 1.1 us.  A 64-row matrix takes 36.5 us (37.2 with a move for every broadcast; 39.5 with a wave in turn that handed the column
// over and one that kept the vector, and with loads for rows that are not there).  What a group leaves is worked off by one compute
// unit instead of 16 or 32.
constexpr int DPP_ROR1 = 0x121, DPP_ROR2 = 0x122, DPP_ROR4 = 0x124;

// over the 16 lanes of a row, in every lane, the same bits for every rotation of the values
__device__ inline double ring_sum(double x)
{
    x += dpp<DPP_ROR8>(x);
    x += dpp<DPP_ROR4>(x);
    x += dpp<DPP_ROR2>(x);
    x += dpp<DPP_ROR1>(x);
    return x;
}
__device__ inline double fold_by(bool up, double a, double b, int which)
{
    const double keep = up ? b : a, give = up ? a : b;
    return keep + (which == 8 ? dpp<DPP_ROR8>(give) : which == 4 ? dpp<DPP_HALF_MIRROR>(give) : dpp<DPP_XOR2>(give));
}
// K <= 8 sums over the 16 lanes of a row at once: lane l receives sum number (l >> 3 & 1) | (l >> 2 & 1) << 1 | (l >> 1 & 1) << 2,
// of as many bits as K needs; there may be none of that number
template <int K>
__device__ inline double row_sums(const double (&v)[K], int lane)
{
    constexpr int K1 = (K + 1) / 2, K2 = (K1 + 1) / 2;
    double a[K1], b[K2];
#pragma unroll
    for (int i = 0; i < K1; ++i) a[i] = 2 * i + 1 < K ? fold_by(lane & 8, v[2 * i], v[2 * i + 1 < K ? 2 * i + 1 : 0], 8) : v[2 * i] + dpp<DPP_ROR8>(v[2 * i]);
#pragma unroll
    for (int i = 0; i < K2; ++i)
        b[i] = 2 * i + 1 < K1 ? fold_by(lane & 4, a[2 * i], a[2 * i + 1 < K1 ? 2 * i + 1 : 0], 4) : a[2 * i] + dpp<DPP_HALF_MIRROR>(a[2 * i]);
    const double c = K2 == 1 ? b[0] + dpp<DPP_XOR2>(b[0]) : fold_by(lane & 2, b[0], b[K2 - 1], 2);
    return c + dpp<DPP_XOR1>(c);
}
template <int K>
__device__ inline int row_slot(int lane)
{
    return (lane >> 3 & 1) | (K > 2 ? (lane >> 2 & 1) << 1 : 0) | (K > 4 ? (lane >> 1 & 1) << 2 : 0);
}

struct TriOne {
    double a[TS][TS];
    double x[TS], v[TS], wv[TS];     // column k; the last step's vectors, which the matrix has still to be updated with
    struct Step { double2 at[ONE + 256]; };                      // A y and column k + 1, and places for sums that are none
    struct Kept { double tau, diagonal, beta; };
    struct Scratch { Step step[2]; Kept kept[ONE]; };            // (by step parity)
    Step* shared;                    // [2]
    Kept* kept;
    int lane, wave, col, row;        // column and row of slot 0
    int off, first;                  // row i here is row i - off of the matrix; the first that is reduced here
    int k_first;                     // the first step
    bool keeps;                      // this lane keeps an entry of every vector, see kept_entry
    Global<double> kept_row;         // where its entry of the last step's belongs

    template <int S>
    __device__ __forceinline__ void steps(int& k, const StepStore& store)
    {
        constexpr int L = TS - S, S1 = S + 1 < TS ? S + 1 : S;
        const int k_end = min(16 * S + 16, ONE - 2);
        // where this lane's sum over a row goes (one that is none: to a place of its own)
        const int t = row_slot<L>(lane);
        const int sum_at = (lane & (L > 4 ? 1 : L > 2 ? 3 : L > 1 ? 7 : 15)) == 0 && t < L ? 16 * (S + t) + row : ONE + (int)threadIdx.x;
        for (; k < k_end; ++k) {
            const int k1 = k + 1;
            const bool next = S + 1 < TS && k1 == 16 * S1;       // row k + 1 is the first of slot S + 1
            Step* sh = shared + (k & 1);
            double sum[L], y[TS], sq = 0.0;
#pragma unroll
            for (int s = S; s < TS; ++s) {
                here(v[s]);
                here(wv[s]);
            }
            wait_for_broadcasts();
#pragma unroll
            for (int s = S; s < TS; ++s) {
                here(v[s]);
                here(wv[s]);
            }
#pragma unroll
            for (int s = S; s < TS; ++s) {
#pragma unroll
                for (int b = S; b < TS; ++b) sub_lane_product<0>(a[s][b], v[s], wv[b]);
#pragma unroll
                for (int b = S; b < TS; ++b) sub_lane_product<0>(a[s][b], wv[s], v[b]);
            }
            // column k + 1 of the matrix: of every row the lane that has that column
            if (col == (k1 & 15)) {
#pragma unroll
                for (int s = S; s < TS; ++s) sh->at[16 * s + row].y = next ? a[s][S1] : a[s][S];
            }
#pragma unroll
            for (int b = S; b < TS; ++b) {
                y[b] = b > S + 1 || 16 * b + col > k1 ? x[b] : 0.0;
                sq = fma(y[b], y[b], sq);
            }
            const double sig2 = ring_sum(sq);
            const int from = (k1 - 4 * wave) & 15;               // the lane of row 0 that has column k + 1
            const double alpha = lane_value(next ? x[S1] : x[S], from);
            double beta, v0, tau;
            householder(alpha, sig2, beta, v0);
            tau = householder_tau(sig2, v0);
#pragma unroll
            for (int r = 0; r < L; ++r) {
                sum[r] = 0.0;
#pragma unroll
                for (int b = S; b < TS; ++b) sum[r] = fma(a[S + r][b], y[b], sum[r]);
            }
            sh->at[sum_at].x = row_sums<L>(sum, lane);
            // the last step's vector, for the way back
            const double entry = kept_entry<S>();
            if (keeps && k > k_first) *kept_row = entry;
            kept_row += k > k_first ? store.N : 0;
#pragma unroll
            for (int b = S; b < TS; ++b) v[b] = b <= S + 1 && 16 * b + col == k1 ? v0 : y[b];
            here(tau);
            __syncthreads();
            double2 pc[TS];
            const double q1 = sh->at[k1].x, c1 = sh->at[k1].y;
#pragma unroll
            for (int b = S; b < TS; ++b) pc[b] = sh->at[16 * b + col];
            __builtin_amdgcn_sched_barrier(0);
            if (wave == (k & 3) && lane < 16 && col == (k & 15)) kept[k] = Kept{tau, x[S], beta};
            double p[TS], gamma = 0.0;
#pragma unroll
            for (int b = S; b < TS; ++b) {
                p[b] = fma(v0, pc[b].y, pc[b].x);
                if (b == S && 16 * b + col <= k) p[b] = 0.0;
                gamma = fma(v[b], p[b], gamma);
            }
            gamma = ring_sum(gamma) * (tau * (0.5 * tau));
            const double wk1 = fma(-gamma, v0, tau * fma(v0, c1, q1));
#pragma unroll
            for (int b = S; b < TS; ++b) {
                wv[b] = fma(-gamma, v[b], tau * p[b]);
                x[b] = fma(-wv[b], v0, fma(-v[b], wk1, pc[b].y));
            }
        }
    }
    // entries of v at the thread's rows: that of row slot 4 h + b in lane 4 b + h of the row of lanes, where a broadcast can be let in by
    // fours of lanes; zeros in what is finished
    template <int S, int H, int B = 0>
    __device__ __forceinline__ void let_in(double& e) const
    {
        if constexpr (4 * H + B >= S) e = row_lane<0, 1 << B>(e, v[4 * H + B]);
        if constexpr (B < 3) let_in<S, H, B + 1>(e);
    }
    template <int S>
    __device__ inline double kept_entry() const
    {
        static_assert(TS == 8, "two fours of slots");
        double low = 0.0, high = 0.0;
        if constexpr (S < 4) let_in<S, 0>(low);
        let_in<S, 1>(high);
        return lane & 1 ? high : low;
    }
    template <int S>
    __device__ __forceinline__ void phases(int& k, const StepStore& store)
    {
        steps<S>(k, store);
        if constexpr (S + 1 < TS) phases<S + 1>(k, store);
    }

    __device__ __forceinline__ void run(const DirectMat& m, Scratch& lds)
    {
        const StepStore store(m);
        const int N = store.N;
        shared = lds.step;
        kept = lds.kept;
        lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        row = 4 * wave + (lane >> 4);
        col = (row + lane) & 15;
        off = ONE - N;
        first = N > ONE ? ONE - TAIL : off;
        int k = N > ONE ? first : off + m.pad;
        // (slots in front of the first are never used, and not loaded: 2 of 37 us for a matrix of 64 rows)
        const Global<const double> C = global((const double*)m.C);
        const bool whole = first == 0;
#pragma unroll
        for (int b = 0; b < TS; ++b) {
            const int c = 16 * b + col - off;
#pragma unroll
            for (int s = 0; s < TS; ++s) a[s][b] = whole || (s >= TS / 2 && b >= TS / 2) ? C[(size_t)(16 * s + row - off) * N + c] : 0.0;
            x[b] = whole || b >= TS / 2 ? C[(size_t)(k - off) * N + c] : 0.0;
            v[b] = wv[b] = 0.0;
        }
        double scale = 1.0;                                      // (larger matrices were scaled by their group)
        if (off >= 0) {
            int expo, zeros;
            scale = scale_of<ONE / 64>(m, off, lane, expo, zeros);
            if (threadIdx.x == 0) {
                m.st[DS_EXP] = expo;
                m.st[DS_ZERO_ROWS] = zeros;
            }
        }
#pragma unroll
        for (int b = 0; b < TS; ++b) {
#pragma unroll
            for (int s = 0; s < TS; ++s) a[s][b] *= scale;
            x[b] *= scale;
        }
        k_first = k;
        // (with zeros in what is finished: a vector is read in pairs of 64 entries)
        const bool pair = first > 0 && !(N / 64 & 1);
        const int number = 16 * (4 * (lane & 3) + (lane >> 2 & 3)) + row;
        keeps = (lane & 3) < TS / 4 && (pair || number >= first);
        kept_row = store.refl + ((size_t)(k - off) * N + number) - off;
        if (first == 0) phases<0>(k, store);
        else phases<TS / 2>(k, store);
        {
            const double entry = kept_entry<TS - 1>();           // (by all lanes: one that is not active has nothing to give)
            if (keeps) *kept_row = entry;
        }
        // what is left: the last 2 x 2 block
        if (row == 15) {
            const double vr = row_lane<0>(v[TS - 1]), wr = row_lane<0>(wv[TS - 1]);
            const double d1 = fma(-wr, v[TS - 1], fma(-vr, wv[TS - 1], a[TS - 1][TS - 1]));
            if (col == 15) {
                store.td[2 * N - 1] = d1;
                store.od[N - 2] = x[TS - 1];
                store.td[2 * N - 2] = fmax(x[TS - 1] * x[TS - 1], OD2_MIN);
            }
            if (col == 14) {
                store.tau[N - 2] = 0.0;
                store.td[2 * N - 3] = x[TS - 1];
            }
        }
        __syncthreads();
        if (k_first + (int)threadIdx.x < ONE - 2) {
            const Kept& e = kept[k_first + threadIdx.x];
            store.put(k_first + (int)threadIdx.x - off, e.tau, e.diagonal, e.beta);
        }
    }
};

// The reduction by one workgroup that waits for nobody: the same steps on the matrix in memory, which nothing needs
// afterwards, from `have` rows on (all of them, if there are no more) until `left` are left.  Two passes over what is left of it per
// step: 4 ms for 200 rows, 42 for 512, 83 for 640.
__device__ __forceinline__ void tri_alone(const DirectMat& m, int have, int left, double* lds)
{
    constexpr int C = MAX_R / 64;
    double *const v = lds, *const p = lds + MAX_R;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), N = m.nt * TILE;
    const StepStore store(m);
    const Global<double> A = global(m.C);
    const bool whole = have >= N;
    int expo = 0, zeros = 0;
    const double scale = whole ? scale_of<C>(m, MAX_R - N, lane, expo, zeros) : 1.0;
    auto load = [&](int i, double (&row)[C]) {                   // row i, lane l: columns l, l + 64, ..; zeros past the end
#pragma unroll
        for (int c = 0; c < C; ++c) row[c] = 64 * c < N ? A[(size_t)i * N + lane + 64 * c] : 0.0;
    };
    __syncthreads();
    if (whole) {
        for (int e = tid; e < N * N; e += 256) A[e] *= scale;
    } else {                                                     // the update that the last step's vectors still owe
        const Global<const double> last = global((const double*)m.half) + HALFWAY;
        for (int e = tid; e < HALFWAY * HALFWAY; e += 256) {
            const int i = e / HALFWAY, j = e % HALFWAY;
            const Global<double> at = A + (size_t)(N - HALFWAY + i) * N + N - HALFWAY + j;
            *at = fma(-last[HALFWAY + i], last[j], fma(-last[i], last[HALFWAY + j], *at));
        }
    }
    __syncthreads();
    for (int k = whole ? m.pad : N - have; k < N - left; ++k) {
        double x[C], sq = 0.0;
        load(k, x);
#pragma unroll
        for (int c = 0; c < C; ++c) sq = lane + 64 * c > k + 1 ? fma(x[c], x[c], sq) : sq;
        double beta, v0;
        const double sig2 = wave_sum(sq);
        householder(A[(size_t)k * N + k + 1], sig2, beta, v0);
        const double tau = householder_tau(sig2, v0);
        if (wave == 0) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int i = lane + 64 * c;
                const double vi = i > k + 1 ? x[c] : i == k + 1 ? v0 : 0.0;
                v[i] = vi;
                if (i < N) store.refl[(size_t)k * N + i] = vi;
            }
            if (lane == 0) store.put(k, tau, A[(size_t)k * N + k], beta);
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < C; ++c) x[c] = v[lane + 64 * c];     // (0 up to k)
        for (int i = k + 1 + wave; i < N; i += 4) {
            double row[C], sum = 0.0;
            load(i, row);
#pragma unroll
            for (int c = 0; c < C; ++c) sum = fma(row[c], x[c], sum);
            sum = wave_sum(sum);
            if (lane == 0) p[i] = tau * sum;
        }
        __syncthreads();
        double w[C], gamma = 0.0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int i = lane + 64 * c;
            w[c] = i > k && i < N ? p[i] : 0.0;
            gamma = fma(x[c], w[c], gamma);
        }
        gamma = wave_sum(gamma) * (0.5 * tau);
#pragma unroll
        for (int c = 0; c < C; ++c) w[c] = fma(-gamma, x[c], w[c]);
        for (int i = k + 1 + wave; i < N; i += 4) {
            const double vi = v[i], wi = fma(-gamma, vi, p[i]);
            double row[C];
            load(i, row);
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (lane + 64 * c > k && 64 * c < N) A[(size_t)i * N + lane + 64 * c] = fma(-wi, x[c], fma(-vi, w[c], row[c]));
        }
        __syncthreads();
    }
    if (left == HALFWAY)
        for (int i = tid; i < HALFWAY; i += 256) {
            m.half[i] = A[(size_t)(N - HALFWAY) * N + N - HALFWAY + i];
            m.half[HALFWAY + i] = m.half[2 * HALFWAY + i] = 0.0;
        }
    if (whole && tid == 0) {
        m.st[DS_EXP] = expo;
        m.st[DS_ZERO_ROWS] = zeros;
    }
}

__device__ __forceinline__ void tri_end(const DirectMat& m, TriEnd end, int have, int left, double2* lds)
{
    if (end == TRI_LAST) tri_alone(m, have, left, (double*)lds);
    if (end == TRI_FAILED && (threadIdx.x & 63) == 0) m.st[DS_FAIL] = 1;
}

// work: matrix (below 0: nothing), member of the group, workgroups of the group.
__global__ __launch_bounds__(256, 2) void direct_tridiagonal(const DirectMat* mats, const Work* work, long long start_ticks)
{
    __shared__ double2 lds[2 * MAX_R];
    static_assert(sizeof(lds) >= sizeof(TriOne::Scratch), "one workgroup's");
    const Work wk = work[blockIdx.x];
    if (wk.mat < 0) return;
    const DirectMat& m = mats[wk.mat];
    TriEnd end = TRI_DONE;
    switch (m.cls) {
        case CLS_64:
        case CLS_128: { TriOne t; t.run(m, *(TriOne::Scratch*)lds); } break;
        case CLS_256: { Tri<4, 4, 64> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); } break;
        case CLS_512:
            if (wk.b == 32) { Tri<8, 4, 128> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); }
            else { Tri<8, 8, 64> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); }
            break;
        default: { Tri<10, 5, 128> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); } break;
    }
    tri_end(m, end, MAX_R, TAIL, lds);
}

// For calls whose groups share compute units, where the issue of all the waves counts and not one step's chain: groups of eight
// workgroups, twelve rows to a wave, for up to HALFWAY rows or for what direct_tridiagonal_half left of more.  Every wave works the
// vectors out for itself, so half of the waves save half of that; and 64 groups have their places at once (75 MB of the 128 MB
// of registers are matrix), where 32 of 512 rows have.  64 x (512 x 4608): 1510 -> 670 us for the first 128 steps, in two turns as
// before, + 655 for the others (700 with registers in scratch memory).  Handing over at 320 rows 30 us more, at 256 70.
__global__ __launch_bounds__(256, 2) void direct_tridiagonal_few(const DirectMat* mats, const Work* work, long long start_ticks)
{
    __shared__ double2 lds[2 * MAX_R];
    const Work wk = work[blockIdx.x];
    if (wk.mat < 0) return;
    const DirectMat& m = mats[wk.mat];
    constexpr int W = 4 * FEW_WGS;
    TriEnd end = TRI_DONE;
    if (m.cls <= CLS_128) { TriOne t; t.run(m, *(TriOne::Scratch*)lds); }
    else if (wk.b > FEW_WGS) {
        if (m.cls == CLS_512) { Tri<8, 4, 128> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); }
        else { Tri<10, 5, 128> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); }
    }
    else if (m.cls == CLS_256) { Tri<4, 256 / W, W> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); }
    else { Tri<HALFWAY / 64, HALFWAY / W, W> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); }
    tri_end(m, end, wk.b > FEW_WGS ? MAX_R : HALFWAY, TAIL, lds);
}

// The larger ones of such a call, down to HALFWAY rows.
__global__ __launch_bounds__(256, 2) void direct_tridiagonal_half(const DirectMat* mats, const Work* work, long long start_ticks)
{
    __shared__ double2 lds[2 * MAX_R];
    const Work wk = work[blockIdx.x];
    if (wk.mat < 0) return;
    const DirectMat& m = mats[wk.mat];
    TriEnd end = TRI_DONE;
    if (m.cls <= CLS_128) { TriOne t; t.run(m, *(TriOne::Scratch*)lds); }
    else if (m.cls == CLS_512) { Tri<8, 8, 64, HALFWAY> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); }
    else { Tri<10, 5, 128, HALFWAY> t; end = t.run(m, wk.a, wk.b, start_ticks, lds); }
    tri_end(m, end, MAX_R, HALFWAY, lds);
}

// What the groups left; one workgroup per matrix.
__global__ __launch_bounds__(256, 1) void direct_tail(const DirectMat* mats)
{
    __shared__ TriOne::Scratch lds;
    if (mats[blockIdx.x].r <= ONE) return;
    TriOne t;
    t.run(mats[blockIdx.x], lds);
}

// ------------------------------------------------------------------------------------------------
// Probabilities, draw, message header; one workgroup per matrix
// ------------------------------------------------------------------------------------------------
// A thread has `per` neighbouring values.  The same test as in block_algorithm1; the tail sums are formed from the small end, over a
// row of 16 lanes through shifts, over the 16 rows of the workgroup one by one.
// Bound: latency, most of it that of a launch and of two loads behind each other.  The draws, which know nothing of the values, are
// made while those are on their way, once, and three barriers are left of seventeen: 64 rows 7.6 -> 4.4 us, the ResNet-18 layers
// 11.0 -> 6.1.
__global__ __launch_bounds__(256) void direct_select(const DirectMat* mats, double s, u64 seed, int* flags)
{
    constexpr int PER = (MAX_R + 255) / 256;
    __shared__ double row_sum[16], tail_at[4];
    __shared__ int first_at[4], kept_in[4];
    const DirectMat& m = mats[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row = tid >> 4, r = m.r;
    const int per = (r + 255) / 256, lo = min(r, tid * per), n = min(r, lo + per) - lo;
    const double l0 = m.lam[0], last = m.lam[r - 1 - min(m.st[DS_ZERO_ROWS], r - 1)];
    const int half = m.st[DS_EXP] / 2, zeros = m.st[DS_ZERO_ROWS], failed = m.st[DS_FAIL];
    double lam[PER];
    float u[PER], key[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) lam[k] = m.lam[min(lo + k, r - 1)];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = lo + k;
        u[k] = 0.0f;
        if (k < per) {
            const u32x4 rnd = philox4x32_10((u64)(i >> 2), m.stream_id, seed);
            u[k] = u01((i & 3) == 0 ? rnd.x : (i & 3) == 1 ? rnd.y : (i & 3) == 2 ? rnd.z : rnd.w);
        }
    }
    const double floor = (double)svd::ZERO_REL * l0;
    double mine = 0.0;
#pragma unroll
    for (int k = PER - 1; k >= 0; --k) {
        key[k] = k < n && lam[k] > floor ? (float)ldexp(sqrt(lam[k]), half) : 0.0f;
        mine += (double)key[k];
    }
    mine += dpp<DPP_SHL1>(mine);
    mine += dpp<DPP_SHL2>(mine);
    mine += dpp<DPP_SHL4>(mine);
    mine += dpp<DPP_SHL8>(mine);
    if ((lane & 15) == 0) row_sum[row] = mine;
    __syncthreads();
    double after = 0.0, suffix[PER];
#pragma unroll
    for (int q = 15; q > 0; --q) after += q > row ? row_sum[q] : 0.0;
    after += dpp<DPP_SHL1>(mine);
    int found = r;
    double tail = 0.0;
#pragma unroll
    for (int k = PER - 1; k >= 0; --k) {
        after += (double)key[k];
        suffix[k] = after;
    }
#pragma unroll
    for (int k = PER - 1; k >= 0; --k)
        if (k < n && (double)key[k] * (s - (double)(lo + k)) <= suffix[k]) {
            found = lo + k;
            tail = suffix[k];
        }
    {
        const u64 any = __ballot(found < r);
        const int l = any ? (int)__ffsll((unsigned long long)any) - 1 : 0;
        const int at = __builtin_amdgcn_readlane(found, l);
        const double t = lane_value(tail, l);
        if (lane == 0) {
            first_at[wave] = at;
            tail_at[wave] = t;
        }
    }
    __syncthreads();
    int ns = r;
    double tail_ns = 0.0;
#pragma unroll
    for (int w = 3; w >= 0; --w)
        if (first_at[w] < r) {
            ns = first_at[w];
            tail_ns = tail_at[w];
        }
    float p[PER];
    int pos = 0, total = 0;
    bool kept[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        p[k] = k < n ? alg1_probability(key[k], lo + k, ns, s, tail_ns) : 0.0f;
        kept[k] = k < n && u[k] < p[k];
        const u64 all = __ballot(kept[k]);
        pos += __popcll(all & ((1ull << lane) - 1));
        total += __popcll(all);
        if (k < n && m.sigma_out) m.sigma_out[lo + k] = key[k];
        if (k < n && m.p_out) m.p_out[lo + k] = p[k];
    }
    if (lane == 0) kept_in[wave] = total;
    __syncthreads();
    total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        pos += w < wave ? kept_in[w] : 0;
        total += kept_in[w];
    }
    if (tid == 0) {
        m.report[0] = 1;
        m.report[1] = 2;
        // all of the spectrum above the floor, but for rows of A that are zero themselves; a matrix of zeros has no atoms
        const bool resolved = zeros >= r || last > FLOOR_REL * l0;
        m.st[DS_ACCEPT] = resolved && failed == 0;
        m.st[DS_BROKEN] = failed;
        *m.count = total;
        atomicMax(&flags[FLAG_MAX_SWEEPS], 1);
        if (total > m.capacity) atomicMax(&flags[FLAG_CAPACITY], 1);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (!kept[k]) continue;
        if (pos < m.capacity) {
            const float weight = key[k] / p[k];
            m.idx[pos] = lo + k;
            if (m.w) m.w[pos] = weight;
            m.weight[pos] = weight;
        }
        ++pos;
    }
}

// ------------------------------------------------------------------------------------------------
// Vectors of the shorter side
// ------------------------------------------------------------------------------------------------
// One workgroup of 32 nt threads (a whole number of waves; of the largest matrix of the call) per kept atom.
//
// First the eigenvector of T for the eigenvalue next to lam, by a twisted factorisation: pivots from the top (wave 0) and
// from the bottom (wave 1) as quotients of the characteristic polynomials of the leading and of the trailing blocks,
// twisted where the two meet with the smallest pivot; the Rayleigh quotient corrects lam, and the next round starts
// from there, until the residual is small enough (KEPT_APART).  Then its image under H, a block of 16 reflectors at a time: a thread owns two neighbouring entries of the
// vector and those columns of V; a wave joins in at the first block that reaches its columns.
// Bound: latency.  One atom of 512 rows: a round of 512 steps 8 us, the vector from it 4, N / 16 blocks with one barrier
// each 27: the sums of 16 products over a wave and over the waves, the factor, V from memory (64 KB per block, two blocks
// on their way while one is worked on).  The ResNet-18 layers 51 us, 64 matrices of 512 rows 77, 64 x 576 12.6; from the middle of
// the cell, with two rounds for every atom above the noise, 66, 148 and 17.0; with one round and one workgroup per compute unit 53, 132 and 13.7.
// Work: matrix, slot.
constexpr int VMAX = MAX_R;
constexpr int VEC_THREADS = VMAX / 2;
constexpr int VEC_ROUNDS = 5;    // one as a rule; two to five for atoms that share a cluster with another kept one
constexpr int FLD = RB + 1;      // row stride of a factor in LDS

// What a round leaves.
struct TwistVector {
    double X[VMAX];                          // the vector
    double lam, scale;                       // the Rayleigh quotient; what X is to be multiplied by, 0: another round, negative: not accepted
};
// What a workgroup works out its eigenvector of T from.
struct Twist {
    // T from the top, padding in front, and from the bottom, padding behind (one turn of sixteen: loads run ahead)
    double2 T[2][VMAX + 16];
    double E[VMAX + 1];                      // couplings of the r rows: E[i] between i - 1 and i, zero at both ends
    // characteristic polynomials of the leading blocks ([0], in units of index + 1) and of the trailing ones ([1]), every
    // pair of neighbours in one scale except where `B` holds the first of the pair in the scale of the second
    double P[2][VMAX + 17], B[2][VMAX / 8 + 2];

    // P and B of one direction, by the first row of 16 lanes, all with the same polynomials: lane j has entry j of sixteen of T, from where
    // it is broadcast; the next sixteen are on their way.  Three instructions per step, broadcasts within the products
    // (64 matrices of 512 rows 86 -> 77 us, the ResNet-18 layers 53.5 -> 51.2 against one lane that read every entry from LDS).
    __device__ inline void polynomials(int dir, int n_pad, double lam, int lane)
    {
        const double2* t = T[dir] + lane;
        double* out = P[dir];
        double* bound = B[dir];
        double p0 = 0.0, p1 = 1.0;
        out[0] = 1.0;
        double2 next = *t;
        for (int i = 0; i < n_pad; i += 16) {
            double d = next.y - lam, e = next.x;
            next = t[i + 16];
            broadcasts(d, e);
            double step[16];
            for_lanes([&](auto u) {
                constexpr int U = decltype(u)::value;
                double p2 = 0.0;
                sub_lane_product<U>(p2, e, p0);
                add_lane_product<U>(p2, d, p1);
                step[U] = p1 = (p0 = p1, p2);
                if constexpr (U % 8 == 7) {
                    // the larger of the two to [0.5, 1): 2^(1022 - E), E its exponent as it is stored
                    const unsigned x = max(hi32(p0) & 0x7ff00000u, hi32(p1) & 0x7ff00000u);
                    const double scale = mk64(0u, 0x7fd00000u - x);
                    p0 *= scale;
                    p1 *= scale;
                    step[U] = p1;
                    bound[(i + U) >> 3] = p0;
                }
            });
#pragma unroll
            for (int u = 0; u < 16; ++u) out[i + 1 + u] = step[u];
        }
    }

    // The vector, by one wave: lane l the entries l per .. of it, per <= PER.
    template <int PER>
    __device__ inline void vector(TwistVector& to, int n, int skip, double lambda, double good, const KeptApart& apart, bool last, int lane) const
    {
        // pivots: top = P_{i+1} / P_i, bottom likewise; where they meet with the smallest pivot
        const int per = (n + 63) / 64, i0 = min(n, lane * per), i1 = min(n, i0 + per);
        double d[PER], e_up[PER], e_dn[PER], top[PER], bot[PER], best = 1e300, gamma = 0.0;
        int at = 0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = min(i0 + u, n - 1), s = skip + i, j = n - 1 - i;    // s, j: steps that made them
            d[u] = T[0][s].y;
            e_up[u] = E[i];
            e_dn[u] = E[i + 1];
            top[u] = P[0][s + 1] * reciprocal((s & 7) == 7 ? B[0][s >> 3] : P[0][s]);
            bot[u] = P[1][j + 1] * reciprocal((j & 7) == 7 ? B[1][j >> 3] : P[1][j]);
            const double g = top[u] + bot[u] - (d[u] - lambda);
            if (i0 + u < i1 && fabs(g) < best) { best = fabs(g); gamma = g; at = i; }
        }
        for (int o = 32; o > 0; o >>= 1) {
            const double ob = __shfl_xor(best, o), og = __shfl_xor(gamma, o);
            const int oa = __shfl_xor(at, o);
            if (ob < best || (ob == best && oa < at)) { best = ob; gamma = og; at = oa; }
        }
        // entries from the twist outwards: products of -e_i / top_i downwards and of -e_{i-1} / bottom_i upwards,
        // per lane over its own entries, then over the lanes
        double f[PER], up = 1.0, down = 1.0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = i0 + u;
            const bool before = i < at;
            const double x = (before ? -e_dn[u] : -e_up[u]) * reciprocal(before ? top[u] : bot[u]);
            f[u] = i < i1 && i != at ? x : 1.0;
            down *= before ? f[u] : 1.0;
            up *= before ? 1.0 : f[u];
        }
        double up_before = up, down_after = down;
        for (int o = 1; o < 64; o <<= 1) {
            const double x = __shfl_up(up_before, o), y = __shfl_down(down_after, o);
            if (lane >= o) up_before *= x;
            if (lane + o < 64) down_after *= y;
        }
        up_before = __shfl_up(up_before, 1);
        down_after = __shfl_down(down_after, 1);
        if (lane == 0) up_before = 1.0;
        if (lane == 63) down_after = 1.0;
        double x[PER], sq = 0.0, weight = 0.0, run = up_before;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (i0 + u >= at) run *= f[u];
            x[u] = run;
        }
        run = down_after;
#pragma unroll
        for (int u = PER - 1; u >= 0; --u) {
            if (i0 + u < at) {
                run *= f[u];
                x[u] = run;
            }
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const bool in = i0 + u < i1;
            const double z2 = in ? x[u] * x[u] : 0.0;
            if (in) to.X[i0 + u] = x[u];
            sq += z2;
            weight = fma(z2, fabs(d[u]) + (fabs(e_up[u]) + fabs(e_dn[u])), weight);
        }
        const double norm2 = wave_sum(sq), inv = reciprocal(norm2), size = root(norm2), res = fabs(gamma) * reciprocal(size);    // |T x - lam x| / |x|
        weight = wave_sum(weight) * inv;
        lambda = fma(gamma, inv, lambda);                        // Rayleigh quotient
        // over: the residual is small enough, or it never will be (the eigenvalue was not separated from that of
        // another kept atom, or the factorisation broke down)
        if (lane == 0) {
            to.lam = lambda;
            to.scale = res <= (last ? 100.0 * good : good) && apart.vector(res, weight, lambda) ? reciprocal(size)
                    : last || !apart.possible ? -1.0 : 0.0;
        }
    }
};

// The factors take the place of T and its polynomials, which the rounds have done with by then: 512 rows are 76 KB, two workgroups on a
// compute unit, for calls that have more atoms than compute units (64 matrices of 512 rows, 256 atoms on average, 132 -> 86 us; with the
// factors beside T, asked for at the start, the ResNet-18 layers took 1 us less, 601 rows 1.5).
constexpr int VEC_LDS_MAX = VMAX * FLD * (int)sizeof(double);
static_assert(VEC_LDS_MAX >= (int)sizeof(Twist), "the larger of the two");
inline size_t vec_lds(int max_nt) { return std::max((size_t)max_nt * TILE * FLD * sizeof(double), sizeof(Twist)); }
__global__ __launch_bounds__(VEC_THREADS, 1) void direct_vectors(const DirectMat* mats, const Work* work)
{
    extern __shared__ __attribute__((aligned(16))) double fact[];
    Twist& tw = *(Twist*)fact;
    __shared__ TwistVector tv;
    __shared__ double part[2][VEC_THREADS / 64][RB], red[VEC_THREADS / 64];
    const Work wk = work[blockIdx.x];
    const DirectMat& m = mats[wk.mat];
    const int slot = wk.a, tid = threadIdx.x, lane = tid & 63, n = m.r, nthr = blockDim.x, nw = nthr >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (slot >= min(*m.count, m.capacity)) return;
    const int N = m.nt * TILE, pad = m.pad;
    // its eigenvalue and those of the kept atoms beside it, all three on their way at once (an entry that is not there is
    // not used, whatever it is)
    double own[3], beside[2], lam;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int at = min(max(m.idx[min(max(slot + k - 1, 0), m.capacity - 1)], 0), n - 1);
        own[k] = m.lam[at];
        if (k == 1) {
            lam = m.fine[at];
            beside[0] = at > 0 ? m.lam[at - 1] : 1e300;
            beside[1] = at + 1 < n ? m.lam[at + 1] : -1e300;
        }
    }
    const KeptApart apart(own[1], slot > 0 ? own[0] : -1.0, slot + 1 < min(*m.count, m.capacity) ? own[2] : -1.0,
                          4.0 / (double)(1 << LAM_BITS));
    // A residual of `good` is what the middle of a cell can have and a second round improves to the rounding.  The first round starts from a
    // better value; it is the last where its residual turns the vector by less than 1e-9 (a sixtieth of a unit of fp32; 1.5e-8 and two
    // rounds always have the same errors against LAPACK, 2.5e-8 root mean square, and this one the same times), or where the middle would do.
    const double good = 1e-14 * m.lam[0];
    const double at_once = fabs(lam - own[1]) <= good ? good : fmin(good, 1e-9 * fmin(beside[0] - own[1], own[1] - beside[1]));
    const int first = pad & ~15, n_pad = N - first;
    for (int i = tid; i < n_pad; i += nthr) {
        const doublex2 t = ((Global<const doublex2>)global((const double*)m.td))[first + i];
        tw.T[0][i] = make_double2(t.x, t.y);
        tw.T[1][n_pad - 1 - i].y = t.y;
        tw.T[1][n_pad - i].x = t.x;                              // (the coupling to the entry before comes a step later)
    }
    for (int i = tid; i <= n; i += nthr) tw.E[i] = i > 0 && i < n ? global((const double*)m.od)[pad + i - 1] : 0.0;
    if (tid < 16) {
        tw.T[0][n_pad + tid] = make_double2(0.0, 2.0);
        if (tid > 0) tw.T[1][n_pad + tid].x = 0.0;
        tw.T[1][n_pad + tid].y = 2.0;
    }
    if (tid == 0) tw.T[1][0].x = 0.0;
    __syncthreads();
    for (int round = 0; round < VEC_ROUNDS; ++round) {
        // wave 0 the leading blocks, wave 1 the trailing ones (a workgroup of one wave: both)
        if (lane < 16 && wave < 2) {
            tw.polynomials(wave, n_pad, lam, lane);
            if (nw == 1) tw.polynomials(1, n_pad, lam, lane);
        }
        __syncthreads();
        if (wave == 0) {
            const bool last = round == VEC_ROUNDS - 1;
            const int skip = pad - first;
            const double small = round == 0 ? at_once : good;
            if (n <= 64) tw.vector<1>(tv, n, skip, lam, small, apart, last, lane);
            else if (n <= 128) tw.vector<2>(tv, n, skip, lam, small, apart, last, lane);
            else if (n <= 256) tw.vector<4>(tv, n, skip, lam, small, apart, last, lane);
            else if (n <= 512) tw.vector<8>(tv, n, skip, lam, small, apart, last, lane);
            else tw.vector<VMAX / 64>(tv, n, skip, lam, small, apart, last, lane);
        }
        __syncthreads();
        lam = tv.lam;
        if (tv.scale != 0.0) break;
        __syncthreads();
    }
    // back through H
    const int c0 = 2 * tid;                                      // this thread's entries: c0, c0 + 1
    struct Block { doublex2 v[RB]; };
    // (no branch around the loads: behind one, the wait for an older block would be one for all of them)
    auto fetch = [&](int blk, Block& at) {
        const Global<const char> row = (Global<const char>)(global((const double*)m.refl) + (size_t)max(blk, 0) * RB * N);
        const unsigned offset = 8u * (unsigned)min(c0, N - 2);
#pragma unroll
        for (int j = 0; j < RB; ++j) at.v[j] = *(Global<const doublex2>)(row + (size_t)j * N * 8 + offset);
    };
    const double scale = tv.scale;
    if (tid == 0 && !(scale > 0.0)) {
        m.st[DS_ACCEPT] = 0;
        m.st[DS_BROKEN] = 1;
    }
    double y0 = c0 >= pad && c0 < N ? tv.X[c0 - pad] * scale : 0.0;
    double y1 = c0 + 1 >= pad && c0 < N ? tv.X[c0 + 1 - pad] * scale : 0.0;
    const int last = (N - 3) / RB, first_block = pad / RB;
    auto apply = [&](int b, const Block& at) {
        double prod[RB];
        const double* f = fact + (size_t)b * (RB * FLD) + (lane & 15) * FLD;
#pragma unroll
        for (int j = 0; j < RB; ++j) prod[j] = fma(at.v[j].x, y0, at.v[j].y * y1);
        const double lo = wave_sums<8>((const double(&)[8])prod[0], lane), hi = wave_sums<8>((const double(&)[8])prod[8], lane);
        double(*pt)[RB] = part[b & 1];
        if ((lane & 7) == 0) {
            pt[wave][sum_slot(lane)] = lo;
            pt[wave][8 + sum_slot(lane)] = hi;
        }
        __syncthreads();
        double sum = 0.0;                                        // lane j of a row of 16: the product of vector j with y
#pragma unroll
        for (int w = 0; w < VEC_THREADS / 64; ++w) sum += w < nw ? pt[w][lane & 15] : 0.0;
        double t = 0.0, t_odd = 0.0;
        broadcasts(sum);
        for_lanes([&](auto j) {
            constexpr int J = decltype(j)::value;
            add_lane_product<J>(J & 1 ? t_odd : t, sum, f[J]);
        });
        t += t_odd;
        broadcasts(t);
        for_lanes([&](auto j) {
            constexpr int J = decltype(j)::value;
            sub_lane_product<J>(y0, t, at.v[J].x);
            sub_lane_product<J>(y1, t, at.v[J].y);
        });
        if (c0 >= N) y0 = y1 = 0.0;
    };
    {
        // a wave joins in when its 128 columns are not all finished; the first two blocks from there are on their way by then
        const int start = min(last, (2 * wave + 2) * 64 / RB - 1);
        Block a, c, e;
        fetch(start, a);
        fetch(start - 1, c);
        {
            constexpr int PER = RB;                              // pairs of entries of the factors per thread: N RB / 2, N / 2 threads
            const Global<const doublex2> in = (Global<const doublex2>)global((const double*)m.fact);
            doublex2 x[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) x[u] = in[min(tid + u * nthr, N * RB / 2 - 1)];
            __builtin_amdgcn_sched_barrier(0);                   // (all of them on their way at once, beside the blocks)
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int i = min(tid + u * nthr, N * RB / 2 - 1);
                fact[i / 8 * FLD + 2 * (i & 7)] = x[u].x;
                fact[i / 8 * FLD + 2 * (i & 7) + 1] = x[u].y;
            }
        }
        int b = last;
        for (; b > start; --b) {
            if (lane < RB) part[b & 1][wave][lane] = 0.0;
            __syncthreads();
        }
        for (;;) {
            fetch(b - 2, e);
            apply(b, a);
            if (--b < first_block) break;
            fetch(b - 2, a);
            apply(b, c);
            if (--b < first_block) break;
            fetch(b - 2, c);
            apply(b, e);
            if (--b < first_block) break;
        }
    }
    {
        const double sq = wave_sum(fma(y0, y0, y1 * y1));
        if (lane == 0) red[wave] = sq;
    }
    __syncthreads();
    double sq = 0.0;
    for (int w = 0; w < nw; ++w) sq += red[w];
    const double inv = 1.0 / sqrt(sq);
    const float fold = m.w || m.transposed ? 1.0f : m.weight[slot];  // folded message: the weight goes into U
    const Global<float> out = global(m.transposed ? m.V + (size_t)slot * m.cols : m.U + (size_t)slot * m.rows);
    const Global<double> keep = global(m.u) + (size_t)slot * n;
    if (c0 >= pad && c0 < N) {
        keep[c0 - pad] = y0 * inv;
        out[c0 - pad] = (float)(y0 * inv) * fold;
    }
    if (c0 + 1 >= pad && c0 < N) {
        keep[c0 + 1 - pad] = y1 * inv;
        out[c0 + 1 - pad] = (float)(y1 * inv) * fold;
    }
}

// ------------------------------------------------------------------------------------------------
// Vectors of the longer side: A^T u / sigma, eight kept atoms per turn, summed over the waves four at a time
// ------------------------------------------------------------------------------------------------
constexpr int LONG_COLS = 128;   // positions of the long side per workgroup
constexpr int LONG_GROUP = 8, LONG_PART = 4;   // atoms per turn (a pass over a wide matrix); per sum over the waves

// A message that needs no singular vectors, for a matrix with a kept vector that was not accepted and no iteration behind it:
// the r vectors themselves are an atomic decomposition (A = sum_i |a_i| e_i (a_i / |a_i|)^T), exact, and what is drawn from it
// by Algorithm 1 is an unbiased estimate of A.  Its atoms are sorted by their norms, as singular values are; they are not
// orthogonal to each other.  256 threads of one workgroup.
struct RowAtoms {
    float key[1024];
    int src[1024], count[256];
    Alg1Scratch sc;
    int row[MAX_R];
    float weight[MAX_R];
};
static_assert(MAX_R <= 1024, "keys of one sort");
__device__ inline void row_message(const DirectMat& m, double s, u64 seed, RowAtoms& x, int* flags)
{
    const int tid = threadIdx.x, r = m.r;
    int P = 1;
    while (P < r) P <<= 1;
    __syncthreads();
    for (int i = tid; i < P; i += 256) {
        x.key[i] = i < r ? (float)sqrt(m.diag[m.pad + i]) : -1.0f;
        x.src[i] = i;
    }
    __syncthreads();
    block_sort_desc(x.key, x.src, P);
    const int ns = block_algorithm1(x.key, r, s, x.sc);
    const double tail_ns = x.sc.tail_ns;
    const int per = (r + 255) / 256, lo = min(r, tid * per), hi = min(r, lo + per);
    auto probability = [&](int i) { return alg1_probability(x.key[i], i, ns, s, tail_ns); };
    auto drawn = [&](int i, float p) {
        const u32x4 rnd = philox4x32_10((u64)(i >> 2), m.stream_id, seed);
        return u01((i & 3) == 0 ? rnd.x : (i & 3) == 1 ? rnd.y : (i & 3) == 2 ? rnd.z : rnd.w) < p;
    };
    int mine = 0;
    for (int i = lo; i < hi; ++i) {
        const float p = probability(i);
        if (m.sigma_out) m.sigma_out[i] = x.key[i];
        if (m.p_out) m.p_out[i] = p;
        mine += drawn(i, p);
    }
    x.count[tid] = mine;
    __syncthreads();
    int pos = 0, total = 0;
    for (int t = 0; t < 256; ++t) {
        pos += t < tid ? x.count[t] : 0;
        total += x.count[t];
    }
    for (int i = lo; i < hi; ++i) {
        const float p = probability(i);
        if (!drawn(i, p)) continue;
        if (pos < m.capacity) {
            x.row[pos] = x.src[i];
            x.weight[pos] = x.key[i] / p;
            m.idx[pos] = i;
            if (m.w) m.w[pos] = x.weight[pos];
        }
        ++pos;
    }
    if (tid == 0) {
        *m.count = total;
        if (total > m.capacity) atomicMax(&flags[FLAG_CAPACITY], 1);
    }
    __syncthreads();
    for (int k = 0; k < min(total, m.capacity); ++k) {
        const int row = x.row[k];
        const double inv = 1.0 / sqrt(m.diag[m.pad + row]);
        const float in_u = m.w ? 1.0f : x.weight[k];             // folded message: the weight goes into U
        float* const shorter = m.transposed ? m.V + (size_t)k * m.cols : m.U + (size_t)k * m.rows;
        float* const longer = m.transposed ? m.U + (size_t)k * m.rows : m.V + (size_t)k * m.cols;
        for (int i = tid; i < r; i += 256) shorter[i] = i == row ? (m.transposed ? 1.0f : in_u) : 0.0f;
        for (int c = tid; c < m.M; c += 256) {
            const float g = m.transposed ? m.G[(long long)c * m.ldg + row] : m.G[(long long)row * m.ldg + c];
            longer[c] = (float)((double)g * inv) * (m.transposed ? in_u : 1.0f);
        }
    }
}

// Bound: of a wide matrix the read of the data, once for eight atoms, in rows of 512 bytes (64 x (512 x 4608), 4 atoms on average: 4 at
// a time 187 us, now 157; the ResNet-18 layers, some with more than four, 28.8 -> 20.9).  Of a tall one the read of its 128 positions,
// once for every atom.  512 threads: wave w takes rows w, w + 8, .. of a wide matrix (its 128 positions are two loads of 256 bytes), or
// positions w, w + 8, .. of a tall one.  The first workgroup reports (the host memory that it writes to is far away: it is not to start
// last), and makes the messages of row_message.
__global__ __launch_bounds__(512) void direct_long(const DirectMat* mats, const Work* work, int n_mats, double s, u64 seed,
                                                   int* hint_out, int* flags)
{
    __shared__ __attribute__((aligned(16))) double us[LONG_GROUP][MAX_R];
    __shared__ double red[8][LONG_PART][LONG_COLS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x == 0) {
        static_assert(sizeof(RowAtoms) <= sizeof(us), "made in the place of the vectors");
        __shared__ int broken;
        if (tid >= 256) return;
        if (tid == 0) broken = 0;
        __syncthreads();
        for (int j = tid; j < n_mats; j += 256) {
            const int accepted = mats[j].st[DS_ACCEPT];
            if (!accepted && mats[j].alone) {
                atomicMax(&flags[FLAG_NOCONV], 1);
                if (mats[j].st[DS_BROKEN]) broken = 1;
            }
            if (hint_out) hint_out[HINT_MATS + mats[j].index] = accepted;
        }
        if (hint_out) __threadfence_system();                    // (the host finds the words behind an event without a fence)
        __syncthreads();
        if (hint_out && tid == 0) {
            hint_out[2] = 1;
            __threadfence_system();
        }
        if (broken)
            for (int j = 0; j < n_mats; ++j)
                if (mats[j].alone && mats[j].st[DS_BROKEN]) row_message(mats[j], s, seed, *(RowAtoms*)us, flags);
        return;
    }
    const Work wk = work[blockIdx.x - 1];
    const DirectMat& m = mats[wk.mat];
    const int kept = m.st[DS_BROKEN] ? 0 : min(*m.count, m.capacity), r = m.r, p0 = wk.a * LONG_COLS;
    const Global<const float> G = global(m.G);
    const Global<float> out = global(m.transposed ? m.U : m.V);
    for (int s0 = 0; s0 < kept; s0 += LONG_GROUP) {
        const int ns = min(LONG_GROUP, kept - s0);
        __syncthreads();
        for (int x = tid; x < r; x += 512)
            for (int k0 = 0; k0 < ns; k0 += LONG_PART) {
                double v[LONG_PART];
#pragma unroll
                for (int k = 0; k < LONG_PART; ++k) v[k] = global(m.u)[(size_t)(s0 + min(k0 + k, ns - 1)) * r + x];
#pragma unroll
                for (int k = 0; k < LONG_PART; ++k) us[k0 + k][x] = k0 + k < ns ? v[k] : 0.0;
            }
        __syncthreads();
        // the sums of LONG_PART atoms from k0 on are in `red`
        auto put = [&](int k0) {
            __syncthreads();
            const int k = k0 + tid / LONG_COLS, p = tid % LONG_COLS;
            if (k < ns && p0 + p < m.M) {
                double sum = red[0][k - k0][p];
                if (!m.transposed) {
#pragma unroll
                    for (int q = 1; q < 8; ++q) sum += red[q][k - k0][p];
                }
                const int i = m.idx[s0 + k];
                const double sigma = ldexp(sqrt(m.lam[i]), m.st[DS_EXP] / 2);
                const float fold = m.w || !m.transposed ? 1.0f : m.weight[s0 + k];
                out[(size_t)(s0 + k) * m.M + p0 + p] = (float)(sum / sigma) * fold;
            }
        };
        auto wide = [&](auto number) {
            constexpr int N = decltype(number)::value;
            double acc[N][2];
#pragma unroll
            for (int k = 0; k < N; ++k) acc[k][0] = acc[k][1] = 0.0;
            const int ca = min(p0 + lane, m.M - 1), cb = min(p0 + 64 + lane, m.M - 1);
            for (int i0 = wave; i0 < r; i0 += 8 * 8) {
                float ga[8], gb[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = min(i0 + 8 * u, r - 1);
                    ga[u] = G[(long long)i * m.ldg + ca];
                    gb[u] = G[(long long)i * m.ldg + cb];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = i0 + 8 * u;
                    if (i < r) {
#pragma unroll
                        for (int k = 0; k < N; ++k) {
                            acc[k][0] = fma((double)ga[u], us[k][i], acc[k][0]);
                            acc[k][1] = fma((double)gb[u], us[k][i], acc[k][1]);
                        }
                    }
                }
            }
#pragma unroll
            for (int k0 = 0; k0 < N; k0 += LONG_PART) {
                if (k0 > 0) __syncthreads();
#pragma unroll
                for (int k = 0; k < LONG_PART; ++k) {
                    red[wave][k][lane] = acc[k0 + k][0];
                    red[wave][k][64 + lane] = acc[k0 + k][1];
                }
                put(k0);
            }
        };
        if (!m.transposed) {
            if (ns > LONG_PART) wide(std::integral_constant<int, LONG_GROUP>());
            else wide(std::integral_constant<int, LONG_PART>());
        } else {
            // positions wave, wave + 8, ..: eight at a time, the lanes along the vector
            for (int k0 = 0; k0 < ns; k0 += LONG_PART) {
                if (k0 > 0) __syncthreads();
                for (int h = 0; h < LONG_COLS / 64; ++h) {
                    for (int k = k0; k < min(ns, k0 + LONG_PART); ++k) {
                        double acc[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) acc[u] = 0.0;
                        for (int i = lane; i < r; i += 64) {
                            const double uu = us[k][i];
#pragma unroll
                            for (int u = 0; u < 8; ++u) {
                                const int p = min(p0 + 64 * h + wave + 8 * u, m.M - 1);
                                acc[u] = fma((double)G[(long long)p * m.ldg + i], uu, acc[u]);
                            }
                        }
                        const double sum = wave_sums<8>(acc, lane);
                        if ((lane & 7) == 0) red[0][k - k0][64 * h + wave + 8 * sum_slot(lane)] = sum;
                    }
                }
                put(k0);
            }
        }
    }
}

int class_of(int r)
{
    int c = 0;
    while (64 * CLS_CHUNKS[c] < r) ++c;
    return c;
}

}  // namespace

hipError_t allow_lds()
{
    return hipFuncSetAttribute(reinterpret_cast<const void*>(direct_vectors), hipFuncAttributeMaxDynamicSharedMemorySize, VEC_LDS_MAX);
}

bool eligible(int r) { return r > svd::THIN_R && r <= MAX_R; }

void plan_matrix(Carver& carve, DirectMat& m)
{
    m.nt = (m.r + TILE - 1) / TILE;
    m.pad = m.nt * TILE - m.r;
    m.cls = class_of(m.r);
    const int ntiles = m.nt * (m.nt + 1) / 2;
    // About 320 work items of the Gram product per matrix, none under 128 columns, 64 in matrices of up to three tiles, which leave
    // most of the chip idle (64 x 576: 11.0 -> 5.4 us), at most 64 partial sums; from the shape alone, so that the sums do not
    // depend on what else is in the call.
    const int want = std::max(1, std::min({320 / ntiles, m.M / (ntiles <= 3 ? 64 : 128), 64}));
    m.kchunk = (int)align_up((size_t)(m.M + want - 1) / want, GK);
    m.nchunks = (m.M + m.kchunk - 1) / m.kchunk;
    const size_t N = (size_t)m.nt * TILE;
    m.part = carve.take<double>((size_t)m.nchunks * ntiles * TILE * TILE);
    m.C = carve.take<double>(N * N);
    m.diag = carve.take<double>(N);
    m.refl = carve.take<double>(N * N);
    m.tau = carve.take<double>(N);
    m.td = carve.take<double2>(N);
    m.od = carve.take<double>(N);
    m.fact = carve.take<double>(N * RB);
    m.lam = carve.take<double>(m.r);
    m.fine = carve.take<double>(m.r);
    m.u = carve.take<double>((size_t)m.capacity * m.r);
    m.xch = carve.take<u64>((size_t)XCH * slot_entries(m.cls));
    m.gate = carve.take<u64>(2);
    m.half = carve.take<double>(m.nt * TILE > HALFWAY ? 3 * HALFWAY : 0);
    m.tickets = carve.take<unsigned>(ntiles);
    m.st = carve.take<int>(DS_WORDS);
    m.weight = carve.take<float>(m.capacity);
}

void plan_work(DirectPlan& plan)
{
    size_t steps = 0, longest = 0;                               // of the recurrence, one point for every eigenvalue; of one
    for (const DirectMat& m : plan.mats) {
        steps += (size_t)m.r * m.nt;
        longest = std::max(longest, (size_t)m.nt);
    }
    // Lanes per eigenvalue in the search, which is bound by instruction issue: as many as one wave on every SIMD has, that is
    // as keep all SIMDs busy for one recurrence of the largest matrix (the smaller ones share a SIMD; by the number of eigenvalues
    // alone the ResNet-18 layers would get 8 lanes, half of the SIMDs and two passes more).  64 lanes would
    // take as many passes as 32.
    plan.eig_lanes = 32;
    while (plan.eig_lanes > 4 && steps * plan.eig_lanes > 1024 * 64 * longest) plan.eig_lanes /= 2;
    std::vector<Work> factors;
    std::vector<int> order(plan.mats.size());
    for (size_t j = 0; j < order.size(); ++j) order[j] = (int)j;
    // the longest products first: the last workgroups to start set when the launch ends
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return plan.mats[a].kchunk > plan.mats[b].kchunk; });
    for (int j : order) {
        const DirectMat& m = plan.mats[j];
        for (int ti = 0; ti < m.nt; ++ti)
            for (int tj = ti; tj < m.nt; ++tj) {
                for (int q = 0; q < TILE / SUM_ROWS; ++q) plan.tiles.push_back(Work{j, ti, tj, q});
                for (int c = 0; c < m.nchunks; ++c) plan.gram.push_back(Work{j, ti, tj, c});
            }
        for (int i = 0; i < m.r; i += 256 / plan.eig_lanes) plan.eig.push_back(Work{j, i, 0, 0});
        for (int b = m.pad / RB; b <= (m.nt * TILE - 3) / RB; ++b) factors.push_back(Work{j, b, 0, 0});
        plan.max_nt = std::max(plan.max_nt, m.nt);
        for (int k = 0; k < m.capacity; ++k) plan.vec.push_back(Work{j, k, 0, 0});
        for (int p = 0; p < (m.M + LONG_COLS - 1) / LONG_COLS; ++p) plan.lng.push_back(Work{j, p, 0, 0});
    }
    // (the slots that are filled as a rule are the first of each matrix, and the workgroups of the others are done at once)
    std::stable_sort(plan.vec.begin(), plan.vec.end(), [](const Work& a, const Work& b) { return a.a < b.a; });
    plan.n_eig = plan.eig.size();
    plan.eig.insert(plan.eig.end(), factors.begin(), factors.end());
    // us per encode, by direct_gram / by direct_gram_wide: 512 x 4608 (chunks of 576 columns) with 4032 items 1133 / 1140, 6048
    // 1578 / 1569, 8064 1789 / 1747, 17856 3514 / 3319; 512 x 2048 (256) with 6048 1306 / 1317, 8064 1428 / 1403, 17856 2719 / 2620;
    // 384 x 4608 (320) with 5985 1005 / 1035, 8190 1158 / 1136; 256 x 16384 (512) with 6080 933 / 953, 8320 1154 / 1135.  But 192 x 8192
    // (160) with 8112 586 / 712, 18096 1102 / 1144; 320 x 3072 (160) with 8100 826 / 870; 256 x 4096 (128) with 8320 659 / 766, 17920
    // 1194 / 1254.  Nor beside long chunks, which are then a launch of their own: 30 of 512 x 4608 with 60 of 256 x 2304 (128) 2548 / 2738,
    // with 60 of 512 x 1152 (160) 3954 / 4628; the layers of four ResNet-18 gradients 1326 / 1427, but those of 16 4288 / 4214.
    auto whole = [&](const Work& w) {
        const DirectMat& m = plan.mats[w.mat];
        return m.kchunk >= WIDE_COLUMNS && !m.transposed && m.M % 16 == 0 && (m.pad == 0 || w.a > 0) && m.ldg < 1 << 24;
    };
    if ((size_t)std::count_if(plan.gram.begin(), plan.gram.end(), whole) >= WIDE_MIN) {
        // A die works on the tiles of one chunk of columns of one matrix at a time, whose rows they share; the cheaper tiles
        // on the diagonal at the end, where an item more or less on a SIMD sets when the launch ends.
        std::vector<Work> wide[2];
        for (const Work& w : plan.gram)
            if (whole(w)) wide[w.a == w.b].push_back(w);
        for (auto* list : {&plan.gram, &plan.tiles}) list->erase(std::remove_if(list->begin(), list->end(), whole), list->end());
        for (auto& list : wide) {
            std::stable_sort(list.begin(), list.end(), [](const Work& x, const Work& y) { return x.mat != y.mat ? x.mat < y.mat : x.c < y.c; });
            std::vector<std::array<Work, 4>> fours((list.size() + 3) / 4);
            for (auto& f : fours) f.fill(Work{-1, 0, 0, 0});
            for (size_t k = 0; k < list.size(); ++k) fours[k / 4][k % 4] = list[k];
            deal_to_dies(fours);
            for (const auto& f : fours) plan.gram_wide.insert(plan.gram_wide.end(), f.begin(), f.end());
        }
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return plan.mats[a].r > plan.mats[b].r; });
    // Twice the workgroups for matrices of 257 to 512 rows, if every workgroup of the call has a compute unit to itself then: four of
    // 512 rows and five of 256 480 -> 455 us for the first 384 steps; 64 of 512 rows, where it has not, 1395 -> 2297.  What else runs on
    // the device is not known here: the encode of ResNet-18 takes 881 us alone (16 workgroups: 901), 3310 beside the same
    // encode of another context (2985) and 3.9 ms, one call in ten 4.5 - 5.6, beside 8192^3 products in bf16 (3.0 - 3.8, 3.9).  In 60
    // calls each beside these, fp32 products, long products and copies no group gave up its wait for its workgroups.
    auto large = [](const DirectMat& m) { return m.nt * TILE > HALFWAY; };
    struct { int all = 0, large = 0; } most, usual, few;         // workgroups, by matrix: 32 or 16 for 257 to 512 rows; 32, or 8 up to HALFWAY
    for (const DirectMat& m : plan.mats) {
        const int n = CLS_WGS[m.cls], n_most = m.cls == CLS_512 ? 32 : n, n_few = large(m) ? n_most : std::min(n, FEW_WGS);
        most.all += n_most, usual.all += n, few.all += n_few;
        if (large(m)) usual.large += n, few.large += n_few;
    }
    const bool wide = most.all <= 256;
    // Where that is not so, groups of eight for up to HALFWAY rows if the larger ones have a compute unit per workgroup then, all 32 of
    // them, or if there is no larger one and more than 256 workgroups otherwise: us per encode before / with them, n = 1024: 20 of 256
    // rows 455 / 411, 64 of 256 804 / 640, 17 of 320 587 / 530; six of 512 and six of 256 786 / 735, eight of 512 with ten of 256 and ten of
    // 128 817 / 761, six of 512 and 30 of 256 839 / 794.  Not beside more of the larger ones (eight of 512, 30 of 256, four of 600 and 16
    // of 64 1058 / 1103), nor where every workgroup has its compute unit without (nine of 320 447 / 494).
    // In two launches where the larger ones are more than have their places at once: 17 of 640 1950 / 1765, 28 of 512 and four of 640 1749 /
    // 1546, 33 of 512 1721 / 1706, 48 of 512 1885 / 1875, 96 of 512 3453 / 3180; but ten of 512 811 / 951, 17 of 512 1143 / 1150, nine of 640
    // 1312 / 1359.
    const bool beside = !wide && few.large > 0 && few.large <= 256 && few.all <= 512;
    plan.half = usual.large > 512;
    plan.few = beside || plan.half || (!wide && few.large == 0 && usual.all > 256);
    // Workgroup b runs on die b mod 8: every group goes to the die that has the least to do so far, longest chains first.
    auto deal = [&](std::vector<Work>& list, auto&& workgroups) {
        std::vector<Work> die[8];
        long long load[8] = {0};
        for (int j : order) {
            const int wgs = workgroups(plan.mats[j]);
            int best = 0;
            for (int x = 1; x < 8; ++x)
                if (load[x] < load[best]) best = x;
            for (int g = 0; g < wgs; ++g) die[plan.spread ? (best + g) % 8 : best].push_back(Work{j, g, wgs, 0});
            load[best] += (long long)plan.mats[j].r * wgs;
        }
        size_t most = 0;
        for (const auto& l : die) most = std::max(most, l.size());
        list.assign(8 * most, Work{-1, 0, 0, 0});
        for (int x = 0; x < 8; ++x)
            for (size_t k = 0; k < die[x].size(); ++k) list[8 * k + x] = die[x][k];
    };
    if (plan.half) {
        deal(plan.tri_half, [&](const DirectMat& m) { return large(m) || m.cls <= CLS_128 ? CLS_WGS[m.cls] : 0; });
        deal(plan.tri, [&](const DirectMat& m) { return m.cls <= CLS_128 ? 0 : FEW_WGS; });
    } else if (plan.few) {
        deal(plan.tri, [&](const DirectMat& m) { return large(m) ? 32 : std::min(CLS_WGS[m.cls], FEW_WGS); });
    } else {
        deal(plan.tri, [&](const DirectMat& m) { return m.cls == CLS_512 && wide ? 32 : CLS_WGS[m.cls]; });
    }
}

hipError_t launch(const DirectPlan& plan, const DirectTables& t, double s, uint64_t seed, int* hint_out, int* d_flags, hipStream_t stream,
                  hipEvent_t gram_done, hipEvent_t done)
{
    auto grid = [](const std::vector<Work>& list) { return (unsigned)list.size(); };
    // (who waits for an event that was not recorded would not wait for this call)
    const bool wide_last = !plan.gram_wide.empty();
    if (!plan.gram.empty()) {
        direct_gram<<<grid(plan.gram), 256, 0, stream>>>(t.mats, t.gram);
        const hipError_t rc = launch_recorded(wide_last ? nullptr : gram_done, direct_gram_sum, grid(plan.tiles), 256, 0, stream, t.mats, t.tiles);
        if (rc != hipSuccess) return rc;
    }
    if (wide_last) {
        direct_clear_tickets<<<(unsigned)t.n_mats, 64, 0, stream>>>(t.mats);
        const hipError_t rc = launch_recorded(gram_done, direct_gram_wide, (unsigned)((plan.gram_wide.size() + 3) / 4), 256, 0, stream, t.mats,
                                              t.gram_wide, (int)plan.gram_wide.size());
        if (rc != hipSuccess) return rc;
    }
    if (plan.half) direct_tridiagonal_half<<<grid(plan.tri_half), 256, 0, stream>>>(t.mats, t.tri_half, plan.start_ticks);
    if (plan.few) direct_tridiagonal_few<<<grid(plan.tri), 256, 0, stream>>>(t.mats, t.tri, plan.start_ticks);
    else direct_tridiagonal<<<grid(plan.tri), 256, 0, stream>>>(t.mats, t.tri, plan.start_ticks);
    if (plan.max_nt * TILE > ONE) direct_tail<<<(unsigned)t.n_mats, 256, 0, stream>>>(t.mats);
    launch_eigenvalues(plan, t, stream);
    direct_select<<<(unsigned)t.n_mats, 256, 0, stream>>>(t.mats, s, (u64)seed, d_flags);
    const unsigned vec_threads = (unsigned)align_up((size_t)32 * plan.max_nt, 64);
    direct_vectors<<<grid(plan.vec), vec_threads, vec_lds(plan.max_nt), stream>>>(t.mats, t.vec);
    return launch_recorded(done, direct_long, grid(plan.lng) + 1, 512, 0, stream, t.mats, t.lng, t.n_mats, s, (u64)seed, hint_out, d_flags);
}

}  // namespace direct
}  // namespace atomo
