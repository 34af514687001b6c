// Entry-wise ATOMO (Section 3 of arXiv 1806.04090 with the standard basis: lambda_i = g_i, a_i = e_i)
// and the stand-alone Algorithm 1 entry point.
//
// Algorithm 1 without a sort.  The KKT appendix shows the optimum has the water-filling form
// p_i = min(1, |lambda_i| / tau) with one level tau, tau = (sum of the uncapped |lambda|) / (s - n_s)
// (eq. (p_i)).  With N(v) = #{|lambda| > v} and T(v) = sum of the |lambda| <= v, the function
//     h(v) = v * (s - N(v)) - T(v)
// is continuous, has h <= 0 below tau and h > 0 above it, and an element is capped (p = 1) exactly
// when h(|lambda_i|) > 0 - the same test Algorithm 1 applies along the sorted order.  h can be
// evaluated exactly at bucket edges from a histogram that stores, per bucket of the float bit
// pattern, the element count and the sum of the 24-bit significands (all elements of a bucket share
// their exponent, so this integer sum is exact and independent of summation order).  Three levels of
// 11 + 10 + 10 key bits pin tau down to a single float value; each level is one pass over the data
// that only histograms elements inside the bucket chosen by the previous level.  A level whose
// chosen bucket holds zero or one element already decides everything and the remaining levels are
// skipped on the device.
//
// Sampling and packing.  Coordinate i is kept iff u_i < p_i (Philox stream, float32 compare) and is
// stored as (i, g_i / p_i) in ascending i.  The encoder reads the gradient twice: once for the level-0 histogram, once to
// draw every uniform against the bracket that level 0 leaves for p_i; a long one once, against a bracket that a sample of it
// leaves ("sampled levels").  Whatever may be kept is written down in that pass as
// a record (value and offset), and all that follows reads the records, a hundredth of the gradient: the third level of the
// search, the settling of the few draws inside the bracket, the message.  The l_q encoder (Section 4), whose probabilities
// need only a norm, draws against the exact p and has nothing to settle.
#include <cmath>
#include <vector>

#include "atomo_internal.h"

namespace atomo {

namespace {

constexpr int KEY_BITS = 31, L0_BITS = 11, L1_BITS = 10, L2_BITS = 10;
constexpr int NBUCKET = 1 << L0_BITS;        // the largest level
constexpr int HIST_WGS = 1024;
constexpr unsigned int DIRECT_MAX = 65536;   // elements that a pass adds to the next level's global histogram one by one

// What a level leaves behind: either the final answer or the path to continue on.
struct SolveOut {
    int done;                     // n_s and tail are final
    unsigned int prefix;          // key bits chosen so far (not done)
    unsigned long long n_above;   // elements above the chosen bucket
    double sum_below;             // sum of the elements below it
    unsigned long long n_s;       // done: number of capped elements
    double tail;                  // done: sum of the uncapped magnitudes
    double lo, hi;                // level 0: the edges of the chosen bucket; the water level lies in [lo, hi]
    unsigned int count;           // elements in the chosen bucket
    double sum;                   // their sum
};

// A long gradient's water level is looked for among the values around one that a sample of the gradient predicts ("sampled levels").
// Level 1 is then a histogram of the window of WINDOW_BINS of its buckets; each of the workgroups of the draws, DRAW_WGS at most, counts
// and adds up what it finds below and above the window:
constexpr int WINDOW_BINS = 2048;
constexpr int MAX_SHIFT = 11;
constexpr bool sampled_levels(int steps) { return steps == 16; }
constexpr unsigned int NO_WINDOW = ~0u;
constexpr int DRAW_WGS = 4096;
constexpr int REDO_WGS = 1536;               // of the second draws: what the chip holds at once
constexpr int CONFIRM_WGS = 256;
struct Tally {
    double below, inside;         // sums of the elements below the window and inside
    unsigned int n_in, n_from;    // how many inside, how many inside or above
};

struct EwState {
    unsigned int cnt[3][NBUCKET];
    unsigned long long sig[3][NBUCKET];
    SolveOut lvl[3];              // what each level found (written by one kernel, read by the kernels after it);
                                  // lvl[k].done also when an earlier level already settled everything
    unsigned int ticket[65];      // workgroups of a pass that have finished (the last one solves level 0); zero between calls
    unsigned long long n_s;       // final: number of capped elements
    double tail;                  // final: sum of the uncapped magnitudes
    double budget;                // final: s - n_s
    double ratio;                 // final: budget / tail, +inf if tail == 0
    unsigned int n_open;          // records that ew_settle left to ew_write, see Segments::open
    unsigned int shift;           // sampled levels: key >> shift is the bucket of level 1, as many single keys those of level 2
    unsigned int window;          // sampled levels: first bucket of level 1, NO_WINDOW if the sample does not say
    unsigned int dense;           // sampled levels: many elements are to be expected in the window
    unsigned int redo;            // sampled levels: the water level is not in the window, level 0 has been formed of all elements
};


// value of an integer significand sum for elements whose biased exponent is e
__device__ inline double sig_value(unsigned long long sigsum, unsigned int e)
{
    return ldexp((double)sigsum, (int)(e == 0 ? 1 : e) - 150);
}

__device__ inline unsigned int significand(unsigned int key)
{
    const unsigned int e = key >> 23, mant = key & 0x7FFFFFu;
    return e ? (mant | 0x800000u) : mant;
}

// A call finds histograms of zeros.  Level 2, which ew_settle forms, is cleared by the draws in front of it (probabilities: by the pass that
// forms level 1), levels 0 and 1 by the last kernel of a call (their readers have run by then).  Sampled levels: the first draws clear
// level 0, which ew_confirm may form again, of all elements; where it does it clears level 1, all 2048 buckets of the window, of which the
// draws behind it use 1024 (ew_settle looks at the others too).
__device__ inline void clear_level(EwState* st, int level)
{
    for (int i = blockIdx.x * 256 + threadIdx.x; i < NBUCKET; i += gridDim.x * 256) {
        st->cnt[level][i] = 0u;
        st->sig[level][i] = 0ull;
    }
}

__global__ __launch_bounds__(256) void ew_clear(EwState* st)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < 3 * NBUCKET) { (&st->cnt[0][0])[i] = 0u; (&st->sig[0][0])[i] = 0ull; }
    if (i == 0) {
        for (int k = 0; k < 65; ++k) st->ticket[k] = 0u;
        for (int k = 0; k < 3; ++k) { st->lvl[k].done = 0; st->lvl[k].prefix = 0u; st->lvl[k].n_above = 0ull; st->lvl[k].sum_below = 0.0; }
        st->n_s = 0ull; st->tail = 0.0; st->budget = 0.0; st->ratio = 0.0;
    }
}

// Adds the packed words (hist_body) of a workgroup's histogram to the global one.
template <int LEVEL, int COPIES, int NB, int TPB>
__device__ inline void flush_hist(const unsigned long long* acc, EwState* st)
{
#pragma unroll 1
    for (int b = threadIdx.x; b < NB; b += TPB) {
        unsigned int c = 0u;
        unsigned long long sg = 0ull;
#pragma unroll
        for (int k = 0; k < COPIES; ++k) {
            const unsigned long long w = acc[k * NB + b];
            c += (unsigned int)(w >> 40);
            sg += w & ((1ull << 40) - 1);
        }
        if (c) {
            atomicAdd(&st->cnt[LEVEL][b], c);
            atomicAdd(&st->sig[LEVEL][b], sg);
        }
    }
}

// Level-LEVEL histogram of the elements on the path `prefix`, by the TPB threads of workgroup `self` of `members` (all call):
// accumulated in the LDS array acc (COPIES x NB packed words), then added to the global histogram.
// Zeros may be counted or not: for the search they are not there.
template <int LEVEL, int TPB>
__device__ inline void hist_body(const float* __restrict__ g, long long n, EwState* st, unsigned long long* acc, unsigned int prefix,
                                 unsigned int self, unsigned int members)
{
    // Level 0 sees every element and most of them fall into a few dozen buckets: four copies of the
    // histogram (one per lane mod 4) keep lanes of a wave from queueing on the same LDS word.
    // One 64-bit word per bucket: element count in bits 40.., sum of 24-bit significands below.  A
    // workgroup visits fewer than 2^16 elements (checked by the launcher), so neither field overflows.
    constexpr int COPIES = LEVEL == 0 ? 4 : 1;
    constexpr int NB = LEVEL == 0 ? (1 << L0_BITS) : (1 << L1_BITS);
    constexpr int SHIFT = LEVEL == 0 ? 20 : LEVEL == 1 ? 10 : 0;
    const unsigned int copy = LEVEL == 0 ? (threadIdx.x & (COPIES - 1)) * NB : 0u;
    for (int b = threadIdx.x; b < COPIES * NB; b += TPB) acc[b] = 0ull;
    __syncthreads();

    auto visit = [&](float x) {
        const unsigned int key = __float_as_uint(x) & 0x7FFFFFFFu;
        const unsigned long long word = (1ull << 40) | (unsigned long long)significand(key);
        if (LEVEL == 0) {
            atomicAdd(&acc[copy + (key >> SHIFT)], word);
        } else {
            if ((key >> (SHIFT + (LEVEL == 1 ? L1_BITS : L2_BITS))) == prefix)
                atomicAdd(&acc[(key >> SHIFT) & (NB - 1)], word);
        }
    };

    const bool vec = (((size_t)g) & 15) == 0;
    const long long n4 = n / 4;
    const long long stride = (long long)members * TPB;
    // Four loads in flight per thread: one at a time, the pass is a chain of memory latencies.  Level 0: four neighbours of one bucket are
    // one addition, and none if they are zeros: a gradient that is sparse or of few values queues in a few words of the LDS otherwise, the
    // more so the fewer workgroups there are (encode of three million elements, one in 200 not zero, 36.8 -> 24.6 us, all of one magnitude
    // 34.8 -> 23.4; with 256 workgroups instead of 91 and without this 30.7 and 26.6; normal ones 26.4 -> 26.6, with 256 27.6).
    for (long long q0 = (long long)self * TPB + threadIdx.x; q0 < n4; q0 += 4 * stride) {
        float4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long q = q0 + u * stride;
            if (q < n4) x[u] = vec ? ((const float4*)g)[q] : make_float4(g[4 * q], g[4 * q + 1], g[4 * q + 2], g[4 * q + 3]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (q0 + u * stride >= n4) continue;
            if (LEVEL == 0) {
                const float xs[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
                unsigned int key[4], sum = 0u, some = 0u, apart = 0u;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    key[e] = __float_as_uint(xs[e]) & 0x7FFFFFFFu;
                    sum += significand(key[e]);
                    some |= key[e];
                    apart |= key[e] ^ key[0];
                }
                if (apart >> SHIFT == 0u) {
                    if (some) atomicAdd(&acc[copy + (key[0] >> SHIFT)], (4ull << 40) | (unsigned long long)sum);
                    continue;
                }
            }
            visit(x[u].x); visit(x[u].y); visit(x[u].z); visit(x[u].w);
        }
    }
    for (long long i = n4 * 4 + (long long)self * TPB + threadIdx.x; i < n; i += stride) visit(g[i]);
    __syncthreads();
    flush_hist<LEVEL, COPIES, NB, TPB>(acc, st);
}

// Inclusive prefix sums over the lanes of a wave by DPP moves (a shuffle through LDS takes about ten times as long):
// doubling inside the rows of 16 lanes, then the last lane of a row into the rows behind it.
template <int CTRL, int ROWS>
__device__ inline unsigned int dpp_moved(unsigned int v)
{
    return (unsigned int)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS>
__device__ inline double dpp_moved(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned int lo = dpp_moved<CTRL, ROWS>((unsigned int)u), hi = dpp_moved<CTRL, ROWS>((unsigned int)(u >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <typename V>
__device__ inline V wave_prefix(V v)
{
    v += dpp_moved<0x111, 0xF>(v);                               // row_shr:1, 2, 4, 8
    v += dpp_moved<0x112, 0xF>(v);
    v += dpp_moved<0x114, 0xF>(v);
    v += dpp_moved<0x118, 0xF>(v);
    v += dpp_moved<0x142, 0xA>(v);                               // row_bcast:15 into rows 1 and 3
    v += dpp_moved<0x143, 0xC>(v);                               // row_bcast:31 into rows 2 and 3
    return v;
}
// The value of the lane before; 0 in lane 0.
__device__ inline double lane_before(double v) { return dpp_moved<0x138, 0xF>(v); }           // wave_shr:1

// One level of the search, by the T threads of a workgroup (all must call).
// read(b, cnt, sig) gives a bucket of the level's histogram, of NB (`bins` of them in use); `first` is the number of the first one among
// all of its level, of 2^shift keys each, n_above0 and sum_below0 the path chosen so far (level 0: nothing).  The result goes to `out`
// (LDS or global, visible to the workgroup after the call's last barrier).
// scratch: LDS, (2 T / 64 + 1) x 8 bytes.
template <int LEVEL, int T, int NB, typename READ>
__device__ inline void solve_hist(READ read, double s, unsigned int first, unsigned int shift, int bins, unsigned long long n_above0,
                                  double sum_below0, SolveOut* out, unsigned long long* scratch)
{
    unsigned int* cpart = (unsigned int*)scratch;
    double* spart = (double*)(scratch + T / 64);
    int& best = *(int*)(scratch + 2 * (T / 64));
    constexpr int PER = NB / T;
    static_assert(PER >= 1, "one bucket per thread at least");
    const int tid = threadIdx.x;
    auto bucket_key = [&](int b) -> unsigned int { return (first + (unsigned int)b) << shift; };
    // exponent shared by every element on the chosen path (level 0: part of the bucket index)
    auto bucket_exp = [&](int b) -> unsigned int { return bucket_key(b) >> 23; };
    auto bucket_lo = [&](int b) -> double { return (double)__uint_as_float(bucket_key(b)); };

    // this thread's PER consecutive buckets stay in registers
    unsigned int cnt_r[PER];
    double sum_r[PER];
    unsigned int c_mine = 0u;                                    // (n < 2^32: every count fits)
    double s_mine = 0.0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int b = tid * PER + e;
        unsigned long long sg;
        read(b, cnt_r[e], sg);
        sum_r[e] = sig_value(sg, bucket_exp(b));
        c_mine += cnt_r[e];
        s_mine += sum_r[e];
    }
    __syncthreads();                                             // (the scratch may still be read from a previous call)
    // prefix sums over the threads: in the wave, then over the waves
    const int lane = tid & 63, wave = tid >> 6;
    const unsigned int c_scan = wave_prefix(c_mine);
    const double s_scan = wave_prefix(s_mine);
    if (lane == 63) {
        cpart[wave] = c_scan;
        spart[wave] = s_scan;
    }
    if (tid == 0) best = 0;
    __syncthreads();
    unsigned int c_before = c_scan - c_mine, c_all = 0u;         // counts in buckets owned by earlier threads, by all
    double s_before = lane_before(s_scan), earlier = 0.0;        // sum in buckets owned by earlier threads
#pragma unroll
    for (int w = 0; w < T / 64; ++w) {
        const unsigned int c = cpart[w];
        const double d = spart[w];
        c_all += c;
        c_before += w < wave ? c : 0u;
        earlier += w < wave ? d : 0.0;
    }
    s_before += earlier;
    const unsigned int c_after = c_all - c_before - c_mine;      // counts in buckets owned by later threads

    // h at the lower edge of bucket b:  lo_b * (s - #{elements in buckets >= b}) - sum(buckets < b)
    {
        unsigned int at_or_above = c_after + c_mine;
        double below = s_before;
        int mine_best = -1;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int b = tid * PER + e;
            const double h = bucket_lo(b) * (s - (double)(n_above0 + at_or_above)) - (sum_below0 + below);
            if (h <= 0.0 && b < bins) mine_best = b;
            at_or_above -= cnt_r[e];
            below += sum_r[e];
        }
        // h is monotone: the highest lane of a wave that has one holds the wave's last bucket (64 lanes' atomics on one word
        // would be performed one after the other)
        const unsigned long long have = __ballot(mine_best >= 0);
        if (have && lane == 63 - __builtin_clzll(have)) atomicMax(&best, mine_best);
    }
    __syncthreads();
    const int bs = best;
    if (tid == bs / PER) {                      // the owner of the chosen bucket finishes from its registers
        unsigned int above = c_after;
        double below = s_before;
        unsigned int c = 0;
        double bucket_sum = 0.0;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int b = tid * PER + e;
            if (b > bs) above += cnt_r[e];
            if (b < bs) below += sum_r[e];
            if (b == bs) { c = cnt_r[e]; bucket_sum = sum_r[e]; }
        }
        const unsigned long long n_above = n_above0 + above;
        const double sum_below = sum_below0 + below;
        bool done = false;
        unsigned long long n_s = n_above;
        double tail = sum_below;
        if (c == 0) {
            done = true;
        } else if (c == 1) {
            const double x = bucket_sum;                       // the element itself
            if (x * (s - (double)n_above) - sum_below - x > 0.0) n_s = n_above + 1;
            else tail = sum_below + x;
            done = true;
        } else if (LEVEL == 2) {
            tail = sum_below + bucket_sum;                     // equal elements at the level: uncapped
            done = true;
        }
        out->done = done ? 1 : 0;
        out->count = c;
        out->sum = bucket_sum;
        out->n_s = n_s;
        out->tail = tail;
        out->n_above = n_above;
        out->sum_below = sum_below;
        out->prefix = first + (unsigned int)bs;
        out->lo = bucket_lo(bs);
        out->hi = bs + 1 < NB ? bucket_lo(bs + 1) : __longlong_as_double(0x7FF0000000000000LL);
    }
    __syncthreads();
}

// Level 0 from a histogram in st->cnt / st->sig that other workgroups of the running kernel wrote (atomics): device-scope
// atomic loads instead of plain ones.
__device__ inline void load_bucket0(const EwState* st, int b, unsigned int& cnt, unsigned long long& sig)
{
    cnt = __hip_atomic_load(&st->cnt[0][b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sig = __hip_atomic_load(&st->sig[0][b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int T>
__device__ inline void solve_level0(const EwState* st, double s, SolveOut* out, unsigned long long* scratch)
{
    solve_hist<0, T, 1 << L0_BITS>([&](int b, unsigned int& cnt, unsigned long long& sig) { load_bucket0(st, b, cnt, sig); },
                                   s, 0u, KEY_BITS - L0_BITS, 1 << L0_BITS, 0ull, 0.0, out, scratch);
}

// Levels 1 and 2 from a histogram that an earlier kernel wrote: `bins` <= NB buckets of 2^shift keys, from bucket `first` on.
template <int LEVEL, int T, int NB = 1 << L1_BITS>
__device__ inline void solve_written(const EwState* st, double s, unsigned int first, unsigned int shift, int bins, const SolveOut& in,
                                     SolveOut* out, unsigned long long* scratch)
{
    solve_hist<LEVEL, T, NB>([&](int b, unsigned int& cnt, unsigned long long& sig) {
        cnt = st->cnt[LEVEL][b];
        sig = st->sig[LEVEL][b];
    }, s, first, shift, bins, in.n_above, in.sum_below, out, scratch);
}

// (s - n_s) / tail, or +inf when nothing is left uncapped
__device__ inline double final_ratio(double s, unsigned long long n_s, double tail)
{
    return tail > 0.0 ? (s - (double)n_s) / tail : __longlong_as_double(0x7FF0000000000000LL);
}

// Records what level `level` found; the final quantities once they are known.
__device__ inline void publish(EwState* st, int level, const SolveOut& r, double s)
{
    st->lvl[level] = r;
    if (r.done) {
        st->n_s = r.n_s;
        st->tail = r.tail;
        st->budget = s - (double)r.n_s;
        st->ratio = final_ratio(s, r.n_s, r.tail);
    }
}

// Levels 1 and 2 are solved at the head of the kernel behind the one that wrote the histogram, by each of its workgroups for
// itself: about two microseconds of loads from L2 and scans, where a last workgroup behind a ticket costs the writing kernel
// five to seven (2728 workgroups).  All 256 threads call; out in LDS.

// At the head of a pass that histograms level 2: true if there is something to do for it, with the path in *out.
__device__ inline bool enter_level2(EwState* st, double s, SolveOut* out, unsigned long long* scratch)
{
    const SolveOut in = st->lvl[0];
    if (in.done) return false;
    solve_written<1, 256>(st, s, in.prefix << L1_BITS, L2_BITS, 1 << L1_BITS, in, out, scratch);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish(st, 1, *out, s);
    return !out->done;
}

// Behind it: the final ratio.  SAMPLED: level 1 may have had wider buckets, see EwState::shift.
template <bool SAMPLED = false>
__device__ inline double enter_final(EwState* st, double s, SolveOut* out, unsigned long long* scratch)
{
    if (st->lvl[0].done) return st->ratio;
    const SolveOut in = st->lvl[1];
    if (in.done) return st->ratio;
    if (SAMPLED && st->shift > L2_BITS)
        solve_written<2, 256, 1 << MAX_SHIFT>(st, s, in.prefix << MAX_SHIFT, 0u, 1 << MAX_SHIFT, in, out, scratch);
    else
        solve_written<2, 256>(st, s, in.prefix << L2_BITS, 0u, 1 << L2_BITS, in, out, scratch);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish(st, 2, *out, s);
    return final_ratio(s, out->n_s, out->tail);
}

// True in every thread of the workgroup that finishes last among `members` workgroups numbered from 0 (all threads of every
// workgroup call, at their very end).  The last workgroup may then read what the others added to the global
// histograms, with device-scope atomic loads: every wave first waits until its own atomics have been performed
// (s_waitcnt vmcnt(0): on gfx9 stores and atomics count in vmcnt, and a workgroup barrier alone does not wait for memory
// operations in flight), and device-scope atomics are performed where every compute unit sees them, so no cache
// maintenance is involved.  Nobody waits for anybody: the others simply leave.
// Tickets in two levels (thousands of atomic adds on one address are performed one after the other, about ten
// nanoseconds each): a workgroup counts on word `self` mod 64, the last one of a word counts on word 64.
// ticket: [65] words, zero on entry and zero again when the last workgroup returns.
__device__ inline bool last_workgroup(unsigned int* ticket, unsigned int self, unsigned int members)
{
    __shared__ int last_sh;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");       // (the compiler keeps them in front)
    __builtin_amdgcn_s_waitcnt(0x0F70);                          // vmcnt(0), other counters untouched
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned int slots = min(64u, members), slot = self % slots;
        const unsigned int here = (members - slot + slots - 1) / slots;
        int last = 0;
        if (__hip_atomic_fetch_add(&ticket[slot], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == here - 1)
            last = __hip_atomic_fetch_add(&ticket[64], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == slots - 1;
        last_sh = last;
    }
    __syncthreads();
    if (last_sh && threadIdx.x < 65)                             // for the next call
        __hip_atomic_store(&ticket[threadIdx.x], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return last_sh != 0;
}

// Level 0: the histogram of all elements, and its last workgroup solves the level at once (one launch and one chain of
// dependent loads less than with a kernel for it).
__global__ __launch_bounds__(1024) void ew_hist0_solve0(const float* __restrict__ g, long long n, EwState* st, double s)
{
    __shared__ unsigned long long acc[4 * NBUCKET];
    __shared__ SolveOut out;
    hist_body<0, 1024>(g, n, st, acc, 0u, blockIdx.x, gridDim.x);
    if (!last_workgroup(st->ticket, blockIdx.x, gridDim.x)) return;
    solve_level0<1024>(st, s, &out, acc);                             // (acc is spent: scratch)
    if (threadIdx.x == 0) publish(st, 0, out, s);
}

// ---- sampled levels -----------------------------------------------------------------------------------
// Level 0 only says around which values the water level lies, and 2^20 elements, 32768 pieces of 32 at places that a hash
// chooses, say that well enough: the window of level 1 is the 2^21 or 2^22 values around the level that they give, 6 to 25 % to
// either side.  So the whole gradient is read once for search and draws, where the histogram of level 0 reads it once by itself:
// ew_draw counts and adds up what lies below and above the window, and whether the water level is inside is then an exact
// test.  If it is not (the sample had no part in what counts), or the sample is too scattered to say, level 0 is formed of all elements
// and the draws are made again: more work, the same message.  Two launches more, 4.8 us each where there is nothing to do, and 11 for the
// sample: encode of 34 million elements 82 -> 73 us, 67 million 168 -> 104, 2^28 529 -> 280; where the sample cannot say (40 elements hold
// a tenth of the sum) 66 -> 82, 137 -> 155 and 458 -> 391.
constexpr int SAMPLE = 1 << 20, PIECE = 32, SAMPLE_WGS = 64;
constexpr long long LONG_FROM = 1ll << 25;   // elements from which on segments have 16 steps

__device__ inline double window_edge(unsigned int bucket, unsigned int shift) { return (double)__uint_as_float(bucket << shift); }

// Where the level is by SAMPLE elements with the budget of their share; st->window.  Few workgroups: each adds its hundreds of buckets that
// are not empty to the global histogram one by one.
// How far off that may be is taken from what the workgroups find each for itself, h(level) of its own pieces, every SAMPLE_WGS-th of the
// gradient: neighbours of a gradient may be alike (rows of an embedding of which one in a hundred is not zero), and then the pieces are the
// sample and not their elements.  The window is the wider one, or none, where three deviations ask for it.  With 16384 pieces of 64 taken for
// 2^20 independent elements rows of 64, three in a hundred not zero, gave a level outside the window in one call of four (34 million
// elements 175 us, otherwise 75; now 75).  Pieces of 16 are two cache lines for one and 1 us more, with deviations 0.7 times as large.
// own: [SAMPLE_WGS][NBUCKET / 2], of a workgroup and a pair of buckets the sum of the workgroup's elements below (float) and the number of
// the others.
__global__ __launch_bounds__(1024) void ew_sample(const float* __restrict__ g, long long n, EwState* st, double s, unsigned long long* own)
{
    __shared__ unsigned long long acc[4 * NBUCKET];
    __shared__ SolveOut out;
    __shared__ double spart[16];
    __shared__ unsigned int cpart[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long spacing = n / (SAMPLE / PIECE) / PIECE;      // in pieces
    const bool vec = (((size_t)g) & 15) == 0;
    constexpr int PER = SAMPLE / SAMPLE_WGS / 4096;
    float4 x[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const unsigned int t = u * 1024 + tid, piece = t / (PIECE / 4) * SAMPLE_WGS + blockIdx.x;
        const unsigned int hash = (piece * 0x9E3779B1u) ^ ((piece * 0x85EBCA6Bu) >> 15);
        const long long at = ((long long)piece * spacing + (long long)(((unsigned long long)hash * (unsigned long long)spacing) >> 32)) * PIECE
                             + (t & (PIECE / 4 - 1)) * 4;
        x[u] = vec ? *(const float4*)(g + at) : make_float4(g[at], g[at + 1], g[at + 2], g[at + 3]);
    }
    for (int b = tid; b < 4 * NBUCKET; b += 1024) acc[b] = 0ull;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const float xs[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned int key = __float_as_uint(xs[e]) & 0x7FFFFFFFu;
            if (key) atomicAdd(&acc[(tid & 3) * NBUCKET + (key >> 20)], (1ull << 40) | (unsigned long long)significand(key));
        }
    }
    __syncthreads();
    // a pair of buckets per thread: to the global histogram, and the workgroup's own sums
    static_assert(NBUCKET == 2048, "a pair per thread");
    unsigned int c = 0u;
    double v = 0.0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int b = 2 * tid + e;
        unsigned long long w = 0ull;                             // (16384 elements: the fields of the packed word hold them)
#pragma unroll
        for (int k = 0; k < 4; ++k) w += acc[k * NBUCKET + b];
        const unsigned long long sig = w & ((1ull << 40) - 1);
        if (w) {
            atomicAdd(&st->cnt[0][b], (unsigned int)(w >> 40));
            atomicAdd(&st->sig[0][b], sig);
        }
        c += (unsigned int)(w >> 40);
        v += sig_value(sig, (unsigned int)b >> 3);
    }
    const unsigned int c_scan = wave_prefix(c);
    const double v_scan = wave_prefix(v);
    if (lane == 63) {
        cpart[wave] = c_scan;
        spart[wave] = v_scan;
    }
    __syncthreads();
    unsigned int from = c - c_scan;
    double below = lane_before(v_scan);
    for (int w = 0; w < 16; ++w) {
        from += w < wave ? 0u : cpart[w];
        below += w < wave ? spart[w] : 0.0;
    }
    __hip_atomic_store(&own[blockIdx.x * (NBUCKET / 2) + tid], (unsigned long long)from << 32 | __float_as_uint((float)below), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    if (!last_workgroup(st->ticket, blockIdx.x, gridDim.x)) return;
    const double share = s * ((double)SAMPLE / (double)n);
    solve_level0<1024>(st, share, &out, acc);
    if (wave != 0) return;
    const SolveOut r = out;
    double tau;
    if (r.done) {
        tau = r.tail / (share - (double)r.n_s);
    } else {                                                     // between the edges of the bucket
        const double h_lo = r.lo * (share - (double)(r.n_above + r.count)) - r.sum_below;
        const double h_hi = r.hi * (share - (double)r.n_above) - r.sum_below - r.sum;
        tau = r.lo + (r.hi - r.lo) * (h_lo / (h_lo - h_hi));
    }
    const bool in_range = tau > 0x1p-94 && tau < 0x1p100;        // (not NaN)
    const unsigned int key = in_range ? __float_as_uint((float)tau) : 0u;
    static_assert(MAX_SHIFT == L2_BITS + 1, "a window reaches over one or two buckets of level 0 to either side");
    unsigned int near = 0u;
    unsigned long long sig;
    if (in_range && lane < 5) load_bucket0(st, (int)(key >> 20) + lane - 2, near, sig);
    // sum of min(|x|, level) over each workgroup's elements (those of the pair of buckets count as the level); their variance
    static_assert(SAMPLE_WGS == 64, "one per lane");
    const unsigned long long o = __hip_atomic_load(&own[lane * (NBUCKET / 2) + r.prefix / 2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long all = __hip_atomic_load(&own[lane * (NBUCKET / 2)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const double h = (double)__uint_as_float((unsigned int)o) + tau * (double)(unsigned int)(o >> 32);
    auto total = [](double v) {
        const unsigned long long u = (unsigned long long)__double_as_longlong(wave_prefix(v));
        return __longlong_as_double((long long)((unsigned long long)(unsigned int)__builtin_amdgcn_readlane((int)(u >> 32), 63) << 32 |
                                                (unsigned int)__builtin_amdgcn_readlane((int)u, 63)));
    };
    const double apart = h - total(h) / SAMPLE_WGS, variance = total(apart * apart) * ((double)SAMPLE_WGS / (SAMPLE_WGS - 1));
    const double above = r.done ? (double)r.n_s : (double)r.n_above + (double)r.count * ((r.hi - tau) / (r.hi - r.lo));
    // the window is 2^-4 to 2^-3 of the level to either side, with the wider buckets twice that; 2^32 over its values is a float
    const double off = 3.0 * sqrt(variance);
    auto holds = [&](unsigned int shift) {
        const unsigned int first = (key >> shift) - WINDOW_BINS / 2;
        return off < fmin(tau - window_edge(first, shift), window_edge(first + WINDOW_BINS, shift) - tau) * (share - above);
    };
    // (a budget of nearly all that is not zero: the few smallest elements decide, and a handful of them looks as if it were sure)
    const bool enough = in_range && total((double)(unsigned int)(all >> 32)) - above >= 64.0;
    const bool narrow = enough && holds(L2_BITS);
    near = wave_prefix(narrow && (lane == 0 || lane == 4) ? 0u : near);
    if (lane == 63) {
        const unsigned int shift = narrow ? L2_BITS : MAX_SHIFT;
        st->window = enough && holds(shift) ? (key >> shift) - WINDOW_BINS / 2 : NO_WINDOW;
        st->shift = shift;
        st->dense = (double)near * ((double)n / SAMPLE) > (double)DIRECT_MAX;
    }
}

struct WindowPath {
    double n_above;               // elements above the window
    double sum_below;             // sum of those below
    bool holds;                   // the water level is inside
};

// The tallies of all workgroups, in an order that is always the same.  All 1024 threads call; scratch: LDS, 5 * 16 doubles.
// The sum below is that of its parts to multiples of 2^-52 of a bound, which add up without rounding, and that of the rest, which does not
// count: rounded once (as one sum up to 2e-16 off; by level 0, of sums of buckets that are exact, up to 7e-17 for gradients of several kinds).
__device__ inline WindowPath window_path(const Tally* tally, unsigned int tallies, unsigned int window, unsigned int shift, long long n, double s,
                                         double* scratch)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double lo = window_edge(window, shift), hi = window_edge(window + WINDOW_BINS, shift);
    const unsigned long long bound = (unsigned long long)__double_as_longlong(lo * (double)n);
    const double unit = __longlong_as_double((long long)(((bound >> 52) + 2) << 52));          // more than twice the sum, a power of two
    double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < DRAW_WGS; k += 1024) {
        const Tally t = k + threadIdx.x < tallies ? tally[k + threadIdx.x] : Tally{0.0, 0.0, 0u, 0u};
        const double part = (t.below + unit) - unit;
        v[0] += part; v[1] += t.inside; v[2] += (double)t.n_in; v[3] += (double)t.n_from; v[4] += t.below - part;
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        v[k] = wave_prefix(v[k]);
        if (lane == 63) scratch[k * 16 + wave] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        v[k] = scratch[k * 16];
        for (int w = 1; w < 16; ++w) v[k] += scratch[k * 16 + w];
    }
    WindowPath p;
    p.n_above = v[3] - v[2];
    p.sum_below = v[0] + v[4];
    p.holds = lo * (s - v[3]) - p.sum_below <= 0.0 && hi * (s - p.n_above) - p.sum_below - v[1] > 0.0;
    return p;
}

// Behind the draws: the path into the window, or level 0 of all elements if the water level is not there.  `members` workgroups of
// level 0 on a grid of fewer.
__global__ __launch_bounds__(1024) void ew_confirm(const float* __restrict__ g, long long n, EwState* st, double s, const Tally* tally,
                                                   unsigned int tallies, unsigned int members)
{
    __shared__ unsigned long long acc[4 * NBUCKET];
    __shared__ SolveOut out;
    const unsigned int window = st->window;
    if (window != NO_WINDOW) {
        const WindowPath p = window_path(tally, tallies, window, st->shift, n, s, (double*)acc);
        if (p.holds) {
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                SolveOut& l = st->lvl[0];
                l.done = 0;
                l.n_above = (unsigned long long)p.n_above;
                l.sum_below = p.sum_below;
                st->redo = 0u;
            }
            return;
        }
    }
    for (unsigned int self = blockIdx.x; self < members; self += gridDim.x) {
        __syncthreads();
        hist_body<0, 1024>(g, n, st, acc, 0u, self, members);
    }
    clear_level(st, 1);
    if (!last_workgroup(st->ticket, blockIdx.x, gridDim.x)) return;
    solve_level0<1024>(st, s, &out, acc);
    if (threadIdx.x == 0) {
        publish(st, 0, out, s);
        st->window = out.prefix << L1_BITS;
        st->shift = L2_BITS;
        st->redo = 1u;
    }
}

// p = min(1, |x| (s - n_s) / tail) (eq. (p_i), KKT appendix); `ratio` = (s - n_s) / tail in double,
// or +inf when nothing is left uncapped.  One double multiply and one rounding to float per element.
__device__ inline float ew_probability(float x, double ratio)
{
    const float a = fabsf(x);
    if (a == 0.0f) return 0.0f;
    return fminf(1.0f, (float)((double)a * ratio));
}

// p of every element with the final ratio, by a grid of 256-thread workgroups
__device__ inline void write_p(const float* lam, long long n, double ratio, float* p)
{
    const long long stride = (long long)gridDim.x * 256;
    long long done = 0;
    if (((((size_t)lam) | ((size_t)p)) & 15) == 0) {
        for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < n / 4; q += stride) {
            const float4 x = ((const float4*)lam)[q];
            ((float4*)p)[q] = make_float4(ew_probability(x.x, ratio), ew_probability(x.y, ratio), ew_probability(x.z, ratio),
                                          ew_probability(x.w, ratio));
        }
        done = n / 4 * 4;
    }
    for (long long i = done + (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) p[i] = ew_probability(lam[i], ratio);
}

__global__ __launch_bounds__(256) void ew_write_p(const float* lam, long long n, const EwState* st, float* p)
{
    write_p(lam, n, st->ratio, p);
}

// A load of what is not read again soon: a gradient of several hundred MB that takes its place in the caches drives out what other
// kernels wrote there, and waits for it.
__device__ inline float4 load_once(const float4* p)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 v = __builtin_nontemporal_load((const f4*)p);
    return make_float4(v[0], v[1], v[2], v[3]);
}

__device__ inline float4 load4(const float* g, long long q, long long n, bool vec)
{
    const long long i = q * 4;
    if (vec && i + 3 < n) return ((const float4*)g)[q];
    float4 x;
    x.x = i < n ? g[i] : 0.0f;
    x.y = i + 1 < n ? g[i + 1] : 0.0f;
    x.z = i + 2 < n ? g[i + 2] : 0.0f;
    x.w = i + 3 < n ? g[i + 3] : 0.0f;
    return x;
}

// ---- records ------------------------------------------------------------------------------------------
// A wave owns a segment of the gradient: `steps` float4 per lane, one after the other (step, lane, component = ascending
// index).  The coordinates of the segment that are, or may be, kept are written to the segment's slots in that order: a
// 2-byte word (offset in the segment, and one flag above it) and, for the entry-wise encoder, the 4-byte value.
// The slots are sized for about six times the density of a 1 % message; a segment that holds more is marked and drawn again
// from the gradient wherever its records would be read (same draws, same result), so any distribution is encoded.
constexpr int STEP = 256;                    // elements of a wave per step
constexpr int STEP_BYTES = 288;              // slots per step: 48 entry-wise records, 144 of l_q
constexpr unsigned int OVER = 0x80000000u;   // segment with more candidates than slots
constexpr unsigned int FLAG_BIT = 0x1000u;   // entry-wise: kept for sure; l_q: negative
constexpr unsigned int DROPPED = 0x2000u;    // entry-wise: settled, not kept
constexpr int MAX_GROUP = 64;
constexpr unsigned int COUNTED = 0x80000000u;   // in group_kept: the group's final count, by ew_write
constexpr int SPIN_COUNTED = 1 << 14;        // Segments::spins, about ten milliseconds: never seen

// A record whose draw lies between the bounds that level 1 gives for its p.
struct EwOpen {
    unsigned int i;
    float x;
};

struct Segments {
    unsigned int* count;          // [n_seg] records of a segment; in a group with an OVER among them: kept coordinates | OVER
    unsigned int* group_kept;     // [n_groups] kept coordinates of a group of per_group segments
    unsigned char* slots;
    long long n_seg, n_groups;
    int slot_bytes;               // per segment
    int per_group;
    EwOpen* open;                 // [open_max] the first open records, in any order
    Tally* tally;                 // [DRAW_WGS] sampled levels
    unsigned int open_max;
    int spins;                    // loads of another workgroup's count before it is made anew
};

// Entry-wise records: values first, then the words.
struct Slots {
    float* val;
    unsigned short* word;
    int capacity;
};

__device__ inline Slots ew_slots(const Segments& sg, long long seg)
{
    unsigned char* p = sg.slots + seg * sg.slot_bytes;
    const int cap = sg.slot_bytes / 6 & ~1;
    return Slots{(float*)p, (unsigned short*)(p + 4 * cap), cap};
}

__device__ inline Slots lq_slots(const Segments& sg, long long seg)
{
    return Slots{nullptr, (unsigned short*)(sg.slots + seg * sg.slot_bytes), sg.slot_bytes / 2};
}

// The records of a group, read by a workgroup as one list: before[k] are those ahead of the group's segment k.
struct Group {
    unsigned int before[MAX_GROUP + 1];
    int over;                     // a segment is OVER: none of the group's records is used
};

// All threads call; the group is complete behind the caller's next barrier.
__device__ inline void load_group(const Segments& sg, long long group, Group& gr)
{
    const int lane = threadIdx.x;
    if (lane >= 64) return;
    const long long first = group * sg.per_group;
    const unsigned int c = lane < sg.per_group && first + lane < sg.n_seg ? sg.count[first + lane] : 0u;
    unsigned int v = c & ~OVER;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned int w = __shfl_up(v, o);
        if (lane >= o) v += w;
    }
    gr.before[lane + 1] = v;
    const unsigned long long over = __ballot((c & OVER) != 0u);
    if (lane == 0) { gr.before[0] = 0u; gr.over = over != 0ull; }
}

// Segment of the group that holds record t
__device__ inline int segment_of(const Group& gr, int per_group, unsigned int t)
{
    int k = 0;
    for (int half = per_group >> 1; half > 0; half >>= 1)
        if (gr.before[k + half] <= t) k += half;
    return k;
}

// ballots[e]: lanes with component e in the list.  Position of this lane's first listed component, and how many there are.
__device__ inline unsigned int listed_before(const unsigned long long (&ballots)[4])
{
    unsigned int r = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        r = __builtin_amdgcn_mbcnt_hi((unsigned int)(ballots[e] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)ballots[e], r));
    return r;
}
__device__ inline unsigned int listed_total(const unsigned long long (&ballots)[4])
{
    return (unsigned int)(__popcll(ballots[0]) + __popcll(ballots[1]) + __popcll(ballots[2]) + __popcll(ballots[3]));
}

// r with  p <= fl32(|x| r) 2^-24  for the p = fl32(|x| ratio) of any x but 0 (the product may be NaN there); see ew_draw.  More than zero,
// so that the product is zero only where p is, whatever the level is.
__device__ inline float upper_ratio(double ratio)
{
    return ratio < 1.0e31 ? fmaxf((float)(ratio * 16777216.0 * (1.0 + 4.76837158203125e-07)), __int_as_float(1)) : __int_as_float(0x7f800000);
}
// r with  fl32(|x| r) (1 - 2^-22) 2^-24 <= p  unless p is below the normal range (the product may be beyond 2^24): a ratio of 1e31
// and more, which times 2^24 may be beyond the float range, is bounded by that of 1e31
__device__ inline float lower_ratio(double ratio)
{
    return (float)(fmin(ratio, 1.0e31) * 16777216.0 * (1.0 - 4.76837158203125e-07));
}
// u < p for sure, for the integer u 2^24: fl32(|x| r) (1 - 2^-22) is more.  Less than 2^-100, where p, less by 2^24, may be so far
// below the normal range that it is rounded to zero, is not enough for the u = 0 that it would count for.
__device__ inline bool surely_below(float u, float x, float r)
{
    return u < fmaf(fminf(16777216.0f, fabsf(x) * r), 1.0f - 2.384185791015625e-07f, -7.888609052210118e-31f);
}
__device__ inline unsigned int candidate_bits(const bool (&in)[4])
{
    return (in[0] ? 1u : 0u) | (in[1] ? 2u : 0u) | (in[2] ? 4u : 0u) | (in[3] ? 8u : 0u);
}
// v[e] by selects (an index would send the array through memory)
__device__ inline float pick(const float (&v)[4], int e)
{
    const float v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];
    const float low = (e & 1) ? v1 : v0, high = (e & 1) ? v3 : v2;
    return (e & 2) ? high : low;
}
// Four steps' float4s of a wave, from float4 q0 + lane on.  `whole`: aligned and all inside the gradient (wave-uniform).
template <bool ONCE = false>
__device__ inline void load_steps(const float* __restrict__ g, long long q0, long long n, bool whole, bool vec, float4 (&x)[4])
{
    const int lane = threadIdx.x & 63;
    if (whole) {
        const float4* p = (const float4*)g + q0 + lane;
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = ONCE ? load_once(p + u * 64) : p[u * 64];
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = load4(g, q0 + u * 64 + lane, n, vec);
    }
}

// Calls visit(position, offset in the segment, value, p) for every kept coordinate of a segment, drawn from the gradient
// with the exact ratio; returns their number.  All lanes of the wave call.
template <int STEPS, bool ONCE = false, typename VISIT>
__device__ inline unsigned int draw_segment(const float* __restrict__ g, long long n, long long seg,
                                            unsigned long long stream_id, unsigned long long seed, double ratio, VISIT visit)
{
    const bool vec = (((size_t)g) & 15) == 0;
    const int lane = threadIdx.x & 63;
    // u >= p is decided in single precision wherever p (1 + 2^-21) leaves no doubt; the rest gets the exact p
    const float r_hi = upper_ratio(ratio);
    const bool whole = vec && (seg + 1) * STEPS * STEP <= n;
    unsigned int fill = 0u;                                      // wave-uniform
    for (int j0 = 0; j0 < STEPS; j0 += 4) {
        float4 xv[4];
        const long long q0 = (seg * STEPS + j0) * 64;
        load_steps<ONCE>(g, q0, n, whole, vec, xv);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const u32x4 rnd = philox4x32_10((unsigned long long)((unsigned int)(q0 + u * 64) + lane), stream_id, seed);
            const float xs[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
            const unsigned int rs[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
            bool in[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) in[e] = !((float)(rs[e] >> 8) >= fabsf(xs[e]) * r_hi);
            if (__ballot(in[0] || in[1] || in[2] || in[3]) == 0ull) continue;
            float ps[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ps[e] = ew_probability(xs[e], ratio);
                in[e] = in[e] && u01(rs[e]) < ps[e];
            }
            unsigned long long ballots[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) ballots[e] = __ballot(in[e]);
            unsigned int pos = fill + listed_before(ballots);
            unsigned int left = candidate_bits(in);
            while (__ballot(left != 0u)) {
                if (left) {
                    const int e = __builtin_ctz(left);
                    left &= left - 1;
                    visit(pos++, (unsigned int)((j0 + u) * STEP + lane * 4 + e), pick(xs, e), pick(ps, e));
                }
            }
            fill += listed_total(ballots);
        }
    }
    return fill;
}

// The pass of the entry-wise encoder that draws; the level-0 result is read from st->lvl[0] (the launch before left it there), or the
// window of a sample from st->window.
// After level 0 the water level tau = tail / (s - n_s) is known to lie inside one bucket [lo, hi] of the float bit pattern
// (12.5 % wide), so p_i = min(1, |g_i| / tau) is bracketed for every element, and because rounding is monotone,
// fl(|g_i| / hi) <= p_i <= fl(|g_i| / lo)  holds for the float32 p_i that the final ratio will give.  An element is dropped
// here if u >= p_hi, marked as kept for sure if u < p_lo; what lies between (about 0.12 s elements) is settled by ew_settle and ew_write
// once the remaining levels have fixed tau exactly.  Every element of the chosen bucket has p_hi >= 1 and so a record: level
// 1 is histogrammed here and level 2 from the records.
// Bound by the Philox rounds (18 wide multiplications per four elements) and the read: everything per element that can be left to
// the candidates, one element in fifty, is left to them.  In a long segment a wave queues its candidates until there are 64, one per lane,
// for what they take (bounds, record, histogram): step by step, a handful of lanes goes through that for the others (2^28 elements, 1 %
// kept: 256 -> 244 us; 10 % 310 -> 295; segments of four steps gain nothing).  2^28 elements: 240 us with the sums below the window (10 of
// them), where the histogram of level 0 took 210 and the draws 231.  Read the caches' way the pass takes 300: the decode of the step before
// left its output there.
//
// AFTER says what is known of the level.  EXACT: the bucket of level 0.  SAMPLED: the window of a sample; this pass then adds up
// what lies below it and counts what lies above.  REDO: the bucket again, if the window did not hold the level.
enum After { EXACT, SAMPLED, REDO };
template <int STEPS, After AFTER>
__global__ __launch_bounds__(256) void ew_draw(const float* __restrict__ g, long long n, EwState* st, double s,
                                               unsigned long long stream_id, unsigned long long seed, Segments sg)
{
    constexpr int BINS = AFTER == SAMPLED ? WINDOW_BINS : 1 << L1_BITS;
    __shared__ unsigned long long acc[BINS];                     // packed as in hist_body
    // Candidates of each wave until there are 64 of them: value; the upper 20 bits of its draw and its offset in the segment
    constexpr bool QUEUED = STEPS == 16;
    constexpr unsigned int QUEUE = QUEUED ? 128 : 1;
    __shared__ uint2 queue[4][QUEUE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (AFTER == REDO && !st->redo) return;
    const bool vec = (((size_t)g) & 15) == 0;
    const long long quads = (sg.n_seg + 3) / 4;
    long long seg = (long long)blockIdx.x * 4 + wave;
    bool whole = vec && (seg + 1) * STEPS * STEP <= n;
    if (AFTER == SAMPLED && st->window == NO_WINDOW) {           // (ahead of the loads: 11.7 us of them where it was not, now 5)
        clear_level(st, 0);
        return;                                                  // (the rest is for the next pass)
    }
    float4 xv[4];                                                // (in flight while the search's result arrives)
    load_steps<STEPS == 16>(g, seg * STEPS * 64, n, whole, vec, xv);
    const SolveOut so = st->lvl[0];
    if (AFTER == SAMPLED) clear_level(st, 0);
    clear_level(st, 2);
    if (blockIdx.x == 0 && tid == 0) st->n_open = 0u;
    const unsigned int window = AFTER == SAMPLED ? st->window : so.prefix << L1_BITS, shift = AFTER == SAMPLED ? st->shift : L2_BITS;
    const bool done = AFTER != SAMPLED && so.done != 0;
    const double inf = __longlong_as_double(0x7FF0000000000000LL);
    // Single-precision brackets of the p that the final ratio will give, p = fl32(|g| ratio), scaled by 2^24 like the
    // uniform (an integer below 2^24): with r_lo <= ratio (1 - 2^-22) and r_hi >= ratio (1 + 2^-22),
    // fl32(|g| r_lo) (1 - 2^-22) <= p <= fl32(|g| r_hi) (each rounding moves a value by at most 2^-24 of itself; where
    // |g| r_hi 2^24 underflows, p is zero, and where p is below the normal range see surely_below).  A bracket that is a little wide
    // only sends a few more coordinates to ew_settle, which decides with the exact formula.
    double ratio_lo, ratio_hi;
    if (AFTER == SAMPLED) {
        ratio_lo = 1.0 / window_edge(window + WINDOW_BINS, shift);
        ratio_hi = 1.0 / window_edge(window, shift);
    } else if (done) {
        ratio_lo = ratio_hi = final_ratio(s, so.n_s, so.tail);
    } else {
        ratio_lo = so.hi < inf ? 1.0 / so.hi : 0.0;              // 1 / hi <= ratio <= 1 / lo
        ratio_hi = so.lo > 0.0 ? 1.0 / so.lo : inf;
    }
    const float r_lo = lower_ratio(ratio_lo);
    // The 32 bits w of a draw: (float)w >= fl32(256 |g| r_hi + 512) leaves u 2^24 = w / 256, rounded down, at |g| r_hi or more.  Where
    // 256 r_hi is beyond the float range (water levels of 2^-96 and less; no sampled one) the upper 24 bits are compared with |g| r_hi, and
    // zeros are taken out by hand (0 * infinity, levels below 1e-31).
    const float r_hi = upper_ratio(ratio_hi), r_word = r_hi * 256.0f;
    const bool tiny_level = AFTER != SAMPLED && !(r_word < __int_as_float(0x7f800000));
    // Few elements in the bucket: straight into the global histogram, where they hardly ever meet.  Many: through LDS.
    const bool through_lds = AFTER == SAMPLED ? st->dense != 0u : !done && so.count > DIRECT_MAX;
    const unsigned int first_key = window << shift;
    double below = 0.0, inside = 0.0;                            // this lane's
    unsigned int n_in = 0u, n_from = 0u;
    for (long long quad = blockIdx.x; quad < quads; quad += AFTER == EXACT ? quads : gridDim.x) {
        if (AFTER != EXACT && quad != blockIdx.x) {              // (EXACT has a workgroup for every four segments)
            if (through_lds) __syncthreads();
            seg = quad * 4 + wave;
            whole = vec && (seg + 1) * STEPS * STEP <= n;
            load_steps<STEPS == 16>(g, seg * STEPS * 64, n, whole, vec, xv);
        }
        if (through_lds) {
#pragma unroll 1                                                 // (its addresses would stay in registers through the draws)
            for (int b = tid; b < BINS; b += 256) acc[b] = 0ull;
            __syncthreads();
        }
        if (seg < sg.n_seg) {
            const Slots sl = ew_slots(sg, seg);
            unsigned int fill = 0u, waiting = 0u;                // records written, candidates in the queue, or all if there is none (wave-uniform)
            // an element's place in the search
            auto count = [&](float x) {
                const unsigned int key = __float_as_uint(x) & 0x7FFFFFFFu;
                if (AFTER == SAMPLED && key >= first_key) ++n_from;
                const unsigned int b = (key >> shift) - window;
                if (b < (unsigned int)BINS && !done) {
                    if (AFTER == SAMPLED) {
                        ++n_in;
                        inside += (double)fabsf(x);
                    }
                    if (through_lds) {
                        atomicAdd(&acc[b], (1ull << 40) | (unsigned long long)significand(key));
                    } else {
                        atomicAdd(&st->cnt[1][b], 1u);
                        atomicAdd(&st->sig[1][b], (unsigned long long)significand(key));
                    }
                }
            };
            // a candidate's record, and its place in the search: its draw is u (the queue's is rounded up: less is kept for sure)
            auto record = [&](unsigned int pos, float x, float u, unsigned int offset) {
                if (pos < (unsigned int)sl.capacity) {
                    sl.val[pos] = x;
                    sl.word[pos] = (unsigned short)(offset | (surely_below(u, x, r_lo) ? FLAG_BIT : 0u));
                }
                count(x);
            };
            // the first `number` candidates of the queue, one per lane
            auto records = [&](unsigned int number) {
                lanes_in_order();
                const uint2 c = queue[wave][lane];
                lanes_in_order();                                // (its place is free from here on)
                if ((unsigned int)lane < number)
                    record(fill + lane, __uint_as_float(c.x), (float)((c.y >> 12 << 4) | 15u), c.y & 0xFFFu);
                fill += number;
            };
            auto steps = [&](auto tiny) {
                for (int j0 = 0; j0 < STEPS; j0 += 4) {
                    const long long q0 = (seg * STEPS + j0) * 64;
                    if (j0 > 0) load_steps<STEPS == 16>(g, q0, n, whole, vec, xv);
                    if constexpr (AFTER == SAMPLED) {                // (a NaN is above; beside the draws the sums take twenty registers more)
                        const float edge = __uint_as_float(first_key);
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const float xs[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) below += (double)(fabsf(xs[e]) < edge ? fabsf(xs[e]) : 0.0f);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    // A segment that has run over its slots is drawn again from the gradient: no more draws and records, but the search goes on
                    // (whatever is in it or above is a candidate).  67 million elements, all of them kept: 638 -> 519 us (524 without a sample
                    // and a queue), half of them kept 529 -> 499 (557).
                    if (QUEUED && fill + waiting > (unsigned int)sl.capacity) {
                        for (int u = 0; u < 4; ++u) {
                            const float xs[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (xs[e] != 0.0f) count(xs[e]);
                        }
                        continue;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const u32x4 rnd = philox4x32_10((unsigned long long)((unsigned int)(q0 + u * 64) + lane), stream_id, seed);
                        const float xs[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
                        const unsigned int rs[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
                        bool in[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e)                  // (a NaN is a candidate)
                            in[e] = decltype(tiny)::value ? xs[e] != 0.0f && !((float)(rs[e] >> 8) >= fabsf(xs[e]) * r_hi)
                                                          : !((float)rs[e] >= fmaf(fabsf(xs[e]), r_word, 512.0f));
                        unsigned long long ballots[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) ballots[e] = __ballot(in[e]);
                        if (ballots[0] | ballots[1] | ballots[2] | ballots[3]) {
                            // one candidate per lane and turn: a lane seldom has a second one
                            unsigned int at = waiting + listed_before(ballots), left = candidate_bits(in);
                            waiting += listed_total(ballots);
                            const float rf[4] = {__uint_as_float(rs[0]), __uint_as_float(rs[1]), __uint_as_float(rs[2]), __uint_as_float(rs[3])};
                            for (;;) {
                                do {
                                    if (left && (!QUEUED || at < QUEUE)) {
                                        const int e = __builtin_ctz(left);
                                        left &= left - 1;
                                        const float x = pick(xs, e);
                                        const unsigned int w = __float_as_uint(pick(rf, e)), offset = (unsigned int)((j0 + u) * STEP + lane * 4 + e);
                                        if (QUEUED) queue[wave][at++] = make_uint2(__float_as_uint(x), (w >> 12 << 12) | offset);
                                        else record(at++, x, (float)(w >> 8), offset);
                                    }
                                } while (__ballot(left != 0u && (!QUEUED || at < QUEUE)));
                                if (!QUEUED || waiting < 64u) break;
                                records(64u);
                                queue[wave][lane] = queue[wave][64 + lane];
                                lanes_in_order();
                                waiting -= 64u;
                                at -= 64u;
                            }
                        }
                    }
                }
            };
            // (loops of their own: 11.17 million elements 50.3 us with the decode, 51.7 with a branch in one loop; gradients of 16 and 34 million
            // elements with a level of 1e-30, half of them zeros: 104 -> 63 us and 246 -> 120, with all that is not zero a candidate before)
            if (AFTER != SAMPLED && tiny_level) steps(std::true_type());
            else steps(std::false_type());
            if (QUEUED) records(waiting);
            else fill = waiting;
            if (lane == 0) sg.count[seg] = fill <= (unsigned int)sl.capacity ? fill : OVER;
        }
        if (through_lds) {
            __syncthreads();
            flush_hist<1, 1, BINS, 256>(acc, st);
        }
    }
    if constexpr (AFTER == SAMPLED) {
        __shared__ double sums[2][4];
        __shared__ unsigned int counts[2][4];
        below = wave_prefix(below);
        inside = wave_prefix(inside);
        n_in = wave_prefix(n_in);
        n_from = wave_prefix(n_from);
        if (lane == 63) {
            sums[0][wave] = below;
            sums[1][wave] = inside;
            counts[0][wave] = n_in;
            counts[1][wave] = n_from;
        }
        __syncthreads();
        if (tid == 0)
            sg.tally[blockIdx.x] = Tally{(sums[0][0] + sums[0][1]) + (sums[0][2] + sums[0][3]), (sums[1][0] + sums[1][1]) + (sums[1][2] + sums[1][3]),
                                          counts[0][0] + counts[0][1] + counts[0][2] + counts[0][3],
                                          counts[1][0] + counts[1][1] + counts[1][2] + counts[1][3]};
    }
}

// The uniform of an element
__device__ inline float ew_uniform(unsigned int i, unsigned long long stream_id, unsigned long long seed)
{
    const u32x4 rnd = philox4x32_10((unsigned long long)(i >> 2), stream_id, seed);
    return u01((i & 2) ? ((i & 1) ? rnd.w : rnd.z) : ((i & 1) ? rnd.y : rnd.x));
}

// Solves level 1 and settles the records of a group of segments as far as that goes; level-2 histogram of the elements on the path
// that it chose.  The bucket is 2^-13 of the water level wide, so p is known to that, and of s kept elements about 2^-13 s have their
// draw in between.  Those are listed for ew_write, which solves level 2 at its head; the others are kept or dropped here: one pass over
// the records and one launch less than with a pass for the histogram and another for the draws (11.7 million elements, 1 % kept: 3.8 +
// 4.4 -> 5.8 us; encode and decode of 20,000 elements 25.7 -> 21.6 us, 300,000 26.7 -> 24.6, 11.7 million 53.7 -> 52.3).  Where segments
// have no slots for their candidates their elements are drawn again: sure ones by single-precision bounds (60 million, 20 % kept: 548 ->
// 445 us; 200 million, 15 %: 1308 -> 1275).
// Leaves the count of what is kept for sure.
// Below the normal range the bucket is wider, 2^-139, and where the list would not hold what lies in between (levels up to about
// 6e-39) nothing is settled here.
template <int STEPS>
__global__ __launch_bounds__(256) void ew_settle(const float* __restrict__ g, long long n, EwState* st, double s,
                                                  unsigned long long stream_id, unsigned long long seed, Segments sg)
{
    constexpr bool SAMPLED_LEVELS = sampled_levels(STEPS);
    constexpr int BINS = 1 << (SAMPLED_LEVELS ? MAX_SHIFT : L2_BITS);
    __shared__ unsigned int cnt[BINS];
    __shared__ unsigned long long sig[BINS];
    __shared__ unsigned int wsum[4];
    __shared__ Group gr;
    __shared__ SolveOut out;
    __shared__ unsigned long long scratch[2 * 4 + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long first = (long long)blockIdx.x * sg.per_group;
    load_group(sg, blockIdx.x, gr);
    const SolveOut in = st->lvl[0];
    double ratio_lo, ratio_hi;
    bool search = false;
    bool listed = true;
    unsigned int prefix = 0u, on_path = 0u;
    const unsigned int shift = SAMPLED_LEVELS ? st->shift : L2_BITS;
    if (in.done) {
        ratio_lo = ratio_hi = st->ratio;
    } else {
        if constexpr (SAMPLED_LEVELS)
            solve_written<1, 256, WINDOW_BINS>(st, s, st->window, shift, st->redo ? 1 << L1_BITS : WINDOW_BINS, in, &out, scratch);
        else
            solve_written<1, 256>(st, s, in.prefix << L1_BITS, shift, 1 << L1_BITS, in, &out, scratch);
        if (blockIdx.x == 0 && tid == 0) publish(st, 1, out, s);
        search = out.done == 0;
        prefix = out.prefix;
        on_path = out.count;
        if (search) {                                            // (the sums of the search are good to 2^-40)
            const double lo = (double)__uint_as_float(prefix << shift), hi = (double)__uint_as_float((prefix + 1) << shift);
            ratio_lo = hi < __longlong_as_double(0x7FF0000000000000LL) ? 1.0 / hi * (1.0 - 0x1p-30) : 0.0;
            ratio_hi = lo > 0.0 ? 1.0 / lo * (1.0 + 0x1p-30) : __longlong_as_double(0x7FF0000000000000LL);
            // (about so many draws lie between the bounds, half of the list at most unless the level is below the normal range)
            listed = (s - (double)out.n_above) * (1.0 - ratio_lo / ratio_hi) <= (double)sg.open_max;
        } else {
            ratio_lo = ratio_hi = final_ratio(s, out.n_s, out.tail);
        }
    }
    const bool through_lds = search && on_path > DIRECT_MAX;
    if (through_lds)
        for (int b = tid; b < BINS; b += 256) { cnt[b] = 0u; sig[b] = 0ull; }
    __syncthreads();
    auto visit = [&](float x) {
        const unsigned int key = __float_as_uint(x) & 0x7FFFFFFFu;
        if ((key >> shift) == prefix) {
            const unsigned int b = key & ((1u << shift) - 1u);
            atomicAdd(through_lds ? &cnt[b] : &st->cnt[2][b], 1u);
            atomicAdd(through_lds ? &sig[b] : &st->sig[2][b], (unsigned long long)significand(key));
        }
    };
    // -1 dropped, 1 kept, 0 open and listed
    auto settle = [&](unsigned int i, float x) {
        const float u = ew_uniform(i, stream_id, seed);
        if (!(u < ew_probability(x, ratio_hi))) return -1;
        if (u < ew_probability(x, ratio_lo)) return 1;
        const unsigned int at = atomicAdd(&st->n_open, 1u);
        if (at < sg.open_max) sg.open[at] = EwOpen{i, x};
        return 0;
    };
    unsigned int kept = 0u;                                      // this lane's
    if (!listed) {
        if (gr.over) {
            const long long i1 = min(n, (first + sg.per_group) * STEPS * STEP);
            for (long long i = first * STEPS * STEP + tid; i < i1; i += 256) visit(g[i]);
        } else {
            for (unsigned int t = tid; t < gr.before[MAX_GROUP]; t += 256) {
                const int k = segment_of(gr, sg.per_group, t);
                visit(ew_slots(sg, first + k).val[t - gr.before[k]]);
            }
        }
        if (blockIdx.x == 0 && tid == 0) st->n_open = ~0u;
    } else if (gr.over) {
        const bool vec = (((size_t)g) & 15) == 0;
        const float r_lo = lower_ratio(ratio_lo), r_hi = upper_ratio(ratio_hi);
        for (int k = wave; k < sg.per_group && first + k < sg.n_seg; k += 4) {
            unsigned int sure = 0u;
            const long long seg = first + k;
            const bool whole = vec && (seg + 1) * STEPS * STEP <= n;
            // (a ratio beyond the float range has no bounds in single precision)
            const bool exact = !search && !(ratio_hi < 1.0e31);
            if (exact) {
                const unsigned int c = draw_segment<STEPS>(g, n, seg, stream_id, seed, ratio_hi,
                                                           [](unsigned int, unsigned int, float, float) {});
                sure = lane == 0 ? c : 0u;
            }
            for (int j0 = exact ? STEPS : 0; j0 < STEPS; j0 += 4) {
                float4 xv[4];
                const long long q0 = (seg * STEPS + j0) * 64;
                load_steps(g, q0, n, whole, vec, xv);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const u32x4 rnd = philox4x32_10((unsigned long long)((unsigned int)(q0 + u * 64) + lane), stream_id, seed);
                    const float xs[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
                    const float us[4] = {(float)(rnd.x >> 8), (float)(rnd.y >> 8), (float)(rnd.z >> 8), (float)(rnd.w >> 8)};
                    bool in[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool is_sure = surely_below(us[e], xs[e], r_lo);
                        sure += is_sure ? 1u : 0u;
                        in[e] = !is_sure && !(us[e] >= fabsf(xs[e]) * r_hi);
                        if (search && (q0 + u * 64 + lane) * 4 + e < n) visit(xs[e]);
                    }
                    unsigned int left = candidate_bits(in);
                    while (__ballot(left != 0u)) {
                        if (left) {
                            const int e = __builtin_ctz(left);
                            left &= left - 1;
                            sure += settle((unsigned int)(seg * STEPS * STEP) + (j0 + u) * STEP + lane * 4 + e, pick(xs, e)) > 0 ? 1u : 0u;
                        }
                    }
                }
            }
            kept += sure;
            for (int o = 32; o > 0; o >>= 1) sure += __shfl_xor(sure, o);
            if (lane == 0) sg.count[first + k] = sure | OVER;
        }
    } else {
        for (unsigned int t = tid; t < gr.before[MAX_GROUP]; t += 256) {
            const int k = segment_of(gr, sg.per_group, t);
            const Slots sl = ew_slots(sg, first + k);
            const unsigned int r = t - gr.before[k], word = sl.word[r];
            const float x = sl.val[r];
            if (search) visit(x);
            if (word & FLAG_BIT) {
                ++kept;
            } else {
                const int what = settle((unsigned int)((first + k) * STEPS * STEP) + word, x);
                if (what != 0) sl.word[r] = (unsigned short)(word | (what > 0 ? FLAG_BIT : DROPPED));
                kept += what > 0 ? 1u : 0u;
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) kept += __shfl_xor(kept, o);
    if (lane == 0) wsum[wave] = kept;
    __syncthreads();
    if (tid == 0) sg.group_kept[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    if (through_lds) {
        for (int b = tid; b < BINS; b += 256) {
            if (cnt[b]) {
                atomicAdd(&st->cnt[2][b], cnt[b]);
                atomicAdd(&st->sig[2][b], sig[b]);
            }
        }
    }
}

// The message from the settled records, one group of segments per workgroup, which adds up the counts of all groups before
// its own by itself.  The last group also reports the total.
// LQ: every record is kept, and the message's words are index and sign (bit 31) alone.
// Entry-wise: solves level 2, and draws the records that ew_settle left open with the final ratio, those of the groups before from
// the list.  Without one, or with more of them than it holds, every workgroup draws its group from the gradient, hands the count over
// and waits for those of the groups before, which count theirs before they wait for anybody.  A count that does not come (nothing
// guarantees that workgroups start in order) is made here, so the wait has a bound.  Multiples of 2^-149 up to 200, 40 % kept: 16 million
// 286 us, 268 million 3.6 ms (normal ones 188 us and 1.7 ms; with every workgroup drawing all groups before its own 12.8 and 209 ms).
template <int STEPS, bool LQ>
__global__ __launch_bounds__(256) void ew_write(const float* __restrict__ g, long long n, EwState* st, double s,
                                                unsigned long long stream_id, unsigned long long seed, Segments sg,
                                                long long capacity, unsigned int* __restrict__ idx, float* __restrict__ val,
                                                long long* count_out, int* flags)
{
    __shared__ unsigned long long bsum[4];
    __shared__ unsigned int wsum[2][4];
    __shared__ Group gr;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long first = (long long)blockIdx.x * sg.per_group;
    unsigned long long part = 0ull;
    for (long long i = tid; i < (long long)blockIdx.x; i += 256) part += sg.group_kept[i];
    load_group(sg, blockIdx.x, gr);
    double ratio;
    __shared__ unsigned int more[MAX_GROUP];                     // kept elements of this group's segments that group_kept lacks
    unsigned int n_open = 0u;
    if constexpr (!LQ) {
        __shared__ SolveOut out;
        __shared__ unsigned long long scratch[2 * 4 + 1];
        n_open = st->n_open;
        if (tid < MAX_GROUP) more[tid] = 0u;
        ratio = enter_final<sampled_levels(STEPS)>(st, s, &out, scratch);
        __syncthreads();
    } else {
        ratio = st->ratio;
    }
    // kept by the draw with the final ratio
    auto drawn = [&](unsigned int i, float x) { return ew_uniform(i, stream_id, seed) < ew_probability(x, ratio); };
    const bool listed = n_open <= sg.open_max;
    if constexpr (!LQ) {
        if (listed) {
            for (unsigned int t = tid; t < n_open; t += 256) {
                const EwOpen e = sg.open[t];
                const long long seg = e.i / (STEPS * STEP);
                if (seg < first + sg.per_group && drawn(e.i, e.x)) {
                    if (seg < first) ++part;
                    else atomicAdd(&more[seg - first], 1u);
                }
            }
        } else {
            auto draw = [&](long long seg) {
                return draw_segment<STEPS>(g, n, seg, stream_id, seed, ratio, [](unsigned int, unsigned int, float, float) {});
            };
            for (long long seg = first + wave; seg < min(first + sg.per_group, sg.n_seg); seg += 4) {
                const unsigned int c = draw(seg);
                if (lane == 0) more[seg - first] = c;
            }
            __syncthreads();
            if (wave == 0) {
                unsigned int own = more[lane];
                for (int o = 32; o > 0; o >>= 1) own += __shfl_xor(own, o);
                if (lane == 0) __hip_atomic_store(&sg.group_kept[blockIdx.x], own | COUNTED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            part = 0ull;
            for (unsigned int i0 = wave * 64; i0 < blockIdx.x; i0 += 256) {
                const unsigned int i = min(i0 + lane, blockIdx.x);         // (the own group: counted)
                unsigned int c = 0u;
                unsigned long long missing = __ballot(i < blockIdx.x);
                for (int spins = 0; missing && spins < sg.spins; ++spins) {
                    c = __hip_atomic_load(&sg.group_kept[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    missing = __ballot(!(c & COUNTED) && i < blockIdx.x);
                }
                if ((c & COUNTED) && i < blockIdx.x) part += c & ~COUNTED;
                for (; missing; missing &= missing - 1) {
                    const long long from = (long long)(i0 + __builtin_ctzll(missing)) * sg.per_group;
                    for (long long seg = from; seg < from + sg.per_group; ++seg) {
                        const unsigned int c = draw(seg);
                        if (lane == 0) part += c;
                    }
                }
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) part += __shfl_down(part, o);
    if (lane == 0) bsum[wave] = part;
    __syncthreads();
    unsigned long long base = 0ull;
#pragma unroll
    for (int w = 0; w < 4; ++w) base += bsum[w];
    auto put = [&](unsigned long long pos, unsigned int i, float x, float p) {
        if ((long long)pos < capacity) {
            if (LQ) {
                idx[pos] = i | (x < 0.0f ? 0x80000000u : 0u);
            } else {
                idx[pos] = i;
                val[pos] = x / p;
            }
        }
    };
    if (gr.over) {
        for (int k = wave; k < sg.per_group && first + k < sg.n_seg; k += 4) {
            unsigned long long pos0 = base + gr.before[k];
            const unsigned int i0 = (unsigned int)((first + k) * STEPS * STEP);
            if constexpr (!LQ) {
                if (!listed) pos0 = base;
                for (int j = 0; j < k; ++j) pos0 += more[j];
            }
            draw_segment<STEPS>(g, n, first + k, stream_id, seed, ratio,
                                [&](unsigned int pos, unsigned int off, float x, float p) { put(pos0 + pos, i0 + off, x, p); });
        }
        if (LQ || listed) base += gr.before[MAX_GROUP];
        if constexpr (!LQ)
            for (int j = 0; j < sg.per_group; ++j) base += more[j];
    } else {
        for (unsigned int t0 = 0; t0 < gr.before[MAX_GROUP]; t0 += 256) {
            const unsigned int t = t0 + tid;
            bool keep = false;
            float x = 0.0f;
            unsigned int i = 0u;
            if (t < gr.before[MAX_GROUP]) {
                const int k = segment_of(gr, sg.per_group, t);
                const unsigned int r = t - gr.before[k];
                const Slots sl = LQ ? lq_slots(sg, first + k) : ew_slots(sg, first + k);
                const unsigned int word = sl.word[r];
                x = LQ ? (word & FLAG_BIT ? -1.0f : 1.0f) : sl.val[r];
                keep = LQ || !(word & DROPPED);
                i = (unsigned int)((first + k) * STEPS * STEP) + (word & (FLAG_BIT - 1));
                if (!LQ && keep && !(word & FLAG_BIT)) keep = drawn(i, x);
            }
            if (LQ) {
                if (keep) put(base + t, i, x, 1.0f);
            } else {
                const unsigned long long ballot = __ballot(keep);
                unsigned int (&ws)[4] = wsum[(t0 >> 8) & 1];
                if (lane == 0) ws[wave] = (unsigned int)__popcll(ballot);
                __syncthreads();
                unsigned int ahead = __builtin_amdgcn_mbcnt_hi((unsigned int)(ballot >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((unsigned int)ballot, 0u));
                unsigned int all = 0u;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    if (w < wave) ahead += ws[w];
                    all += ws[w];
                }
                if (keep) put(base + ahead, i, x, ew_probability(x, ratio));
                base += all;
            }
        }
        if (LQ) base += gr.before[MAX_GROUP];
    }
    if (blockIdx.x == gridDim.x - 1 && tid == 0) {
        *count_out = (long long)base;
        if ((long long)base > capacity) atomicMax(&flags[FLAG_CAPACITY], 1);
    }
    if (!LQ) {
        clear_level(st, 0);
        clear_level(st, 1);
    }
}

// The kernels of a gradient below 2^25 elements lie one behind the other: together they are 59 KB of instructions, and apart they drive one
// another out of the 64 KB cache (11.17 million elements with their decode 51.6 us where others lay between, 50.3 so).
template __global__ void ew_draw<4, EXACT>(const float* __restrict__, long long, EwState*, double, unsigned long long, unsigned long long, Segments);
template __global__ void ew_settle<4>(const float* __restrict__, long long, EwState*, double, unsigned long long, unsigned long long, Segments);
template __global__ void ew_write<4, false>(const float* __restrict__, long long, EwState*, double, unsigned long long, unsigned long long, Segments,
                                            long long, unsigned int* __restrict__, float* __restrict__, long long*, int*);

// ---- one workgroup for everything ----------------------------------------------------------------------
// Up to LOCAL_MAX elements are held in the registers of one workgroup: the three levels of the search run in LDS one behind
// the other, without a launch, a ticket or a global atomic between them.  9610 elements: 9.6 us in all (load 0.6, level 0 3.9,
// draws and message 4.2), where five launches took 22.  The draws of one compute unit grow with n: from about 2^15 elements
// on the launches are the cheaper way.
constexpr int LOCAL_T = 1024, LOCAL_PER = 16, LOCAL_MAX = LOCAL_T * LOCAL_PER;

struct LocalScratch {
    unsigned long long hist[4 * NBUCKET];        // packed as in hist_body; four copies at level 0
    unsigned long long solve[2 * (LOCAL_T / 64) + 1];
    SolveOut out;
};

// n_s and tail of the n elements; thread t holds element e * LOCAL_T + t as `key[e]` (bit pattern of the magnitude, ~0 where
// there is none), e < per.  All LOCAL_T threads call; the result is in sc.out for all of them.
__device__ inline void local_water_level(const unsigned int (&key)[LOCAL_PER], int per, double s, LocalScratch& sc)
{
    const int tid = threadIdx.x;
    auto clear = [&](int words) {
        for (int b = tid; b < words; b += LOCAL_T) sc.hist[b] = 0ull;
        __syncthreads();
    };
    auto add = [&](unsigned int b, unsigned int k) {
        atomicAdd(&sc.hist[b], (1ull << 40) | (unsigned long long)significand(k));
    };
    const unsigned int copies = per > 2 ? 4u : 1u, copy = (tid & (copies - 1)) * NBUCKET;
    clear((int)copies * NBUCKET);
#pragma unroll
    for (int e = 0; e < LOCAL_PER; ++e)
        if (e < per && key[e] != ~0u) add(copy + (key[e] >> 20), key[e]);
    __syncthreads();
    solve_hist<0, LOCAL_T, 1 << L0_BITS>([&](int b, unsigned int& cnt, unsigned long long& sig) {
        const unsigned long long w = sc.hist[b];
        cnt = (unsigned int)(w >> 40);
        sig = w & ((1ull << 40) - 1);
        if (copies > 1u) {
#pragma unroll
            for (int c = 1; c < 4; ++c) {
                const unsigned long long v = sc.hist[c * NBUCKET + b];
                cnt += (unsigned int)(v >> 40);
                sig += v & ((1ull << 40) - 1);
            }
        }
    }, s, 0u, KEY_BITS - L0_BITS, 1 << L0_BITS, 0ull, 0.0, &sc.out, sc.solve);
    auto read = [&](int b, unsigned int& cnt, unsigned long long& sig) {
        cnt = (unsigned int)(sc.hist[b] >> 40);
        sig = sc.hist[b] & ((1ull << 40) - 1);
    };
    if (sc.out.done) return;
    SolveOut in = sc.out;
    clear(1 << L1_BITS);
#pragma unroll
    for (int e = 0; e < LOCAL_PER; ++e)
        if (e < per && (key[e] >> 20) == in.prefix) add((key[e] >> 10) & ((1 << L1_BITS) - 1), key[e]);
    __syncthreads();
    solve_hist<1, LOCAL_T, 1 << L1_BITS>(read, s, in.prefix << L1_BITS, L2_BITS, 1 << L1_BITS, in.n_above, in.sum_below, &sc.out, sc.solve);
    if (sc.out.done) return;
    in = sc.out;
    clear(1 << L2_BITS);
#pragma unroll
    for (int e = 0; e < LOCAL_PER; ++e)
        if (e < per && (key[e] >> 10) == in.prefix) add(key[e] & ((1 << L2_BITS) - 1), key[e]);
    __syncthreads();
    solve_hist<2, LOCAL_T, 1 << L2_BITS>(read, s, in.prefix << L2_BITS, 0u, 1 << L2_BITS, in.n_above, in.sum_below, &sc.out, sc.solve);
}

__device__ inline unsigned int magnitude(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }

// Draws and writes the message of a gradient that the workgroup holds: component e of thread t's float4 j is element
// ((j * LOCAL_T + t) * 4 + e).
template <bool LQ>
__device__ inline void local_message(const float (&x)[LOCAL_PER], int n, double ratio, unsigned long long stream_id,
                                     unsigned long long seed, long long capacity, unsigned int* idx, float* val, float* p_out,
                                     long long* count_out, int* flags)
{
    constexpr int W = LOCAL_T / 64;
    __shared__ unsigned int counts[LOCAL_PER / 4 * W + 1];       // kept, then kept before
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float r_hi = upper_ratio(ratio);                       // (see draw_segment)
    unsigned int bits = 0u, before[LOCAL_PER / 4];
#pragma unroll
    for (int j = 0; j < LOCAL_PER / 4; ++j) {
        before[j] = 0u;
        if (j * LOCAL_T * 4 < n) {
            const int q = j * LOCAL_T + tid;
            unsigned long long ballots[4];
            const u32x4 rnd = philox4x32_10((unsigned long long)q, stream_id, seed);
            const unsigned int rs[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
            bool in[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) in[e] = !((float)(rs[e] >> 8) >= fabsf(x[j * 4 + e]) * r_hi);
            if (p_out || __ballot(in[0] || in[1] || in[2] || in[3])) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = ew_probability(x[j * 4 + e], ratio);
                    in[e] = in[e] && u01(rs[e]) < p;
                    if (p_out && q * 4 + e < n) p_out[q * 4 + e] = p;
                }
            }
            bits |= candidate_bits(in) << (4 * j);
#pragma unroll
            for (int e = 0; e < 4; ++e) ballots[e] = __ballot(in[e]);
            before[j] = listed_before(ballots);
            if (lane == 0) counts[j * W + wave] = listed_total(ballots);
        } else if (lane == 0) {
            counts[j * W + wave] = 0u;
        }
    }
    __syncthreads();
    if (wave == 0) {
        static_assert(LOCAL_PER / 4 * W == 64, "one count per lane");
        const unsigned int mine = counts[lane];
        unsigned int v = mine;
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int w = __shfl_up(v, o);
            if (lane >= o) v += w;
        }
        counts[lane] = v - mine;
        if (lane == 63) {
            *count_out = (long long)v;
            if ((long long)v > capacity) atomicMax(&flags[FLAG_CAPACITY], 1);
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < LOCAL_PER / 4; ++j) {
        unsigned int pos = counts[j * W + wave] + before[j], left = (bits >> (4 * j)) & 15u;
        const float xs[4] = {x[j * 4], x[j * 4 + 1], x[j * 4 + 2], x[j * 4 + 3]};
        while (__ballot(left != 0u)) {
            if (left) {
                const int e = __builtin_ctz(left);
                left &= left - 1;
                if ((long long)pos < capacity) {
                    const float xe = pick(xs, e);
                    const unsigned int k = (unsigned int)((j * LOCAL_T + tid) * 4 + e);
                    if (LQ) {
                        idx[pos] = k | (xe < 0.0f ? 0x80000000u : 0u);
                    } else {
                        idx[pos] = k;
                        val[pos] = xe / ew_probability(xe, ratio);
                    }
                }
                ++pos;
            }
        }
    }
}

__device__ inline void local_load(const float* __restrict__ g, int n, float (&x)[LOCAL_PER])
{
    const bool vec = (((size_t)g) & 15) == 0;
#pragma unroll
    for (int j = 0; j < LOCAL_PER / 4; ++j) {
        const float4 v = load4(g, j * LOCAL_T + (int)threadIdx.x, n, vec);
        x[j * 4] = v.x; x[j * 4 + 1] = v.y; x[j * 4 + 2] = v.z; x[j * 4 + 3] = v.w;
    }
}

// The whole entry-wise encoder for n <= LOCAL_MAX.
__global__ __launch_bounds__(LOCAL_T) void ew_encode_local(const float* __restrict__ g, int n, double s, unsigned long long stream_id,
                                                           unsigned long long seed, long long capacity,
                                                           unsigned int* __restrict__ idx, float* __restrict__ val, float* p_out,
                                                           long long* count_out, int* flags)
{
    __shared__ LocalScratch sc;
    float x[LOCAL_PER];
    local_load(g, n, x);
    unsigned int key[LOCAL_PER];
#pragma unroll
    for (int e = 0; e < LOCAL_PER; ++e)
        key[e] = ((e / 4) * LOCAL_T + (int)threadIdx.x) * 4 + e % 4 < n ? magnitude(x[e]) : ~0u;
    local_water_level(key, (n + LOCAL_T * 4 - 1) / (LOCAL_T * 4) * 4, s, sc);
    local_message<false>(x, n, final_ratio(s, sc.out.n_s, sc.out.tail), stream_id, seed, capacity, idx, val, p_out, count_out, flags);
}

// ---- atomo_probabilities --------------------------------------------------------------------------------
struct LocalSeg { long long begin; int n; int pad; };

// First launch: one workgroup per segment of up to LOCAL_MAX elements, start to end, and beside them, on workgroups of their
// own, level 0 of the first longer segment (n_long elements from `lambda_long` on; 0: none).
__global__ __launch_bounds__(LOCAL_T) void prob_first(const float* lam, const LocalSeg* segs, int n_local, double s, float* p,
                                                      const float* lambda_long, long long n_long, EwState* st)
{
    __shared__ LocalScratch sc;
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= n_local) {
        const unsigned int self = blockIdx.x - n_local, members = gridDim.x - n_local;
        hist_body<0, LOCAL_T>(lambda_long, n_long, st, sc.hist, 0u, self, members);
        if (!last_workgroup(st->ticket, self, members)) return;
        solve_level0<LOCAL_T>(st, s, &sc.out, sc.solve);
        if (tid == 0) publish(st, 0, sc.out, s);
        return;
    }
    const LocalSeg seg = segs[blockIdx.x];
    const int per = (seg.n + LOCAL_T - 1) / LOCAL_T;
    float x[LOCAL_PER];
    unsigned int key[LOCAL_PER];
#pragma unroll
    for (int e = 0; e < LOCAL_PER; ++e) {
        const int i = e * LOCAL_T + tid;
        x[e] = i < seg.n ? lam[seg.begin + i] : 0.0f;
    }
#pragma unroll
    for (int e = 0; e < LOCAL_PER; ++e) key[e] = e * LOCAL_T + tid < seg.n ? magnitude(x[e]) : ~0u;
    local_water_level(key, per, s, sc);
    const double ratio = final_ratio(s, sc.out.n_s, sc.out.tail);
#pragma unroll
    for (int e = 0; e < LOCAL_PER; ++e)
        if (e * LOCAL_T + tid < seg.n) p[seg.begin + e * LOCAL_T + tid] = ew_probability(x[e], ratio);
}

// Histograms of levels 1 and 2 of a longer segment, nothing to do where an earlier level settled everything.
template <int LEVEL>
__global__ __launch_bounds__(256) void ew_hist(const float* x, long long n, EwState* st, double s)
{
    __shared__ unsigned long long acc[1 << L1_BITS];
    __shared__ SolveOut out;
    unsigned int prefix;
    if (LEVEL == 1) {
        clear_level(st, 2);
        const SolveOut in = st->lvl[0];
        if (in.done) return;
        prefix = in.prefix;
    } else {
        if (!enter_level2(st, s, &out, acc)) return;
        prefix = out.prefix;
        __syncthreads();
    }
    hist_body<LEVEL, 256>(x, n, st, acc, prefix, blockIdx.x, gridDim.x);
}

// Solves level 2 and writes the probabilities.
__global__ __launch_bounds__(256) void prob_last(const float* lam, long long n, EwState* st, double s, float* p)
{
    __shared__ SolveOut out;
    __shared__ unsigned long long scratch[2 * 4 + 1];
    write_p(lam, n, enter_final(st, s, &out, scratch), p);
    clear_level(st, 0);
    clear_level(st, 1);
}

// ---- l_q quantisation (Section 4) -------------------------------------------------------------------
enum { LQ_MAX = 0, LQ_TWO = 1, LQ_ONE = 2, LQ_POW = 3 };
constexpr int LQ_WGS = 1024;
// From here on both passes read the gradient with load_once.  Up to about 256 MB of gradient and output stay in the last cache from
// pass to pass; beyond that a pass that takes part in it pays for what the decode before left there (norm + draws of 35 million
// elements 26 + 31 us in the caches' way and 28 + 32 so, 50 million 46 + 37 and 37 + 40, 64 million 69 + 44 and 48 + 48, 120 million
// 133 + 96 and 83 + 96).
constexpr long long ONCE_FROM = 42'000'000;

// How |g_i|^q is formed.  PLAIN: q is 1, 2 or infinity.  TABLE: any other q up to TABLE_Q.  POW: beyond.
enum Power { PLAIN, TABLE, POW };
constexpr double TABLE_Q = 4.0;

// a^q of a = 2^e m, 1 <= m < 2, from tables of a workgroup and a short polynomial.  With c_i the middle of the i-th of POWER_PARTS parts of
// [1, 2) and k_i the hardware's reciprocal of it (any number near 1 / c_i would do, as long as it is the same here and there),
//     m^q = k_i^-q (1 + r)^q,   r = m k_i - 1  (exact: 24 + 24 bits),   |r| <= 2^-10,
// and four terms of the binomial series leave out less than C(q, 5) r^5 < 2^-55 for q <= 4.  pow is good to 1.3e-16, this to 5e-16 (root mean
// square 5e-17 and 1.1e-16), without a bias that a sum would show: sums of two million powers, by either, are off by the same 4e-17 to 1.7e-16,
// those of the additions, and norm and p of 3000 to 3 million elements are in every case the float next to the exact value, by either.  A pow takes 970 cycles of a wave: the norm of 10 million elements, q = 1.5,
// 68 -> 19 us, of 100 million 650 -> 111.
constexpr int POWER_PARTS = 512, POWER_LOW = -149, POWER_EXPONENTS = 128 - POWER_LOW + 1;      // 2^-149 to infinity
struct PowerTable {
    double exponent[POWER_EXPONENTS];            // 2^(e q)
    double part[POWER_PARTS];                    // k_i^-q
};
__device__ inline float power_reciprocal(unsigned int part)
{
    return __builtin_amdgcn_rcpf(__uint_as_float(0x3F800000u | (part << 14) | (1u << 13)));
}
// All T threads call; complete behind the caller's next barrier.
template <int T>
__device__ inline void make_power_table(PowerTable& t, double q)
{
    for (int i = threadIdx.x; i < POWER_EXPONENTS + POWER_PARTS; i += T) {
        const bool part = i >= POWER_EXPONENTS;
        const double v = pow(part ? (double)power_reciprocal(i - POWER_EXPONENTS) : ldexp(1.0, i + POWER_LOW), part ? -q : q);
        if (part) t.part[i - POWER_EXPONENTS] = v;
        else t.exponent[i] = i < POWER_EXPONENTS - 1 ? v : __longlong_as_double(0x7FF0000000000000LL);
    }
}
__device__ inline double power_of(double a, double q, const PowerTable& t)
{
    const unsigned long long bits = (unsigned long long)__double_as_longlong(a);
    const unsigned int high = (unsigned int)(bits >> 32), part = (high >> 11) & (POWER_PARTS - 1);
    const int e = min(max((int)(high >> 20) - (1023 + POWER_LOW), 0), POWER_EXPONENTS - 1);      // (0 and NaN: of no use)
    const double m = __longlong_as_double((long long)((bits & 0x000FFFFFFFFFFFFFull) | 0x3FF0000000000000ull));
    const double r = fma(m, (double)power_reciprocal(part), -1.0);
    const double c2 = q * (q - 1.0) * 0.5, c3 = c2 * (q - 2.0) * (1.0 / 3.0), c4 = c3 * (q - 3.0) * 0.25;
    return t.exponent[e] * t.part[part] * fma(r, fma(r, fma(r, fma(r, c4, c3), c2), q), 1.0);
}

// One more element of |g|_q: max |g_i|, or the sum of g_i^2, |g_i| or |g_i|^q in double (pow takes so many registers that it gets kernels
// of its own).
template <Power P>
__device__ inline double lq_add(double acc, float x, int mode, double q, const PowerTable& t)
{
    const double a = (double)fabsf(x);
    if (P == TABLE) return acc + (a > 0.0 ? power_of(a, q, t) : 0.0);
    if (P == POW) return a > 0.0 ? acc + pow(a, q) : acc;
    if (mode == LQ_MAX) return fmax(acc, a);
    if (mode == LQ_TWO) return fma(a, a, acc);
    return acc + a;
}

// Result in thread 0.
template <int T>
__device__ inline double lq_block_reduce(double acc, int mode, double* wpart /* LDS [T / 64] */)
{
    for (int o = 32; o > 0; o >>= 1) {
        const double other = __shfl_down(acc, o);
        acc = mode == LQ_MAX ? fmax(acc, other) : acc + other;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) wpart[threadIdx.x >> 6] = acc;
    __syncthreads();
    double t = wpart[0];
    if (threadIdx.x == 0)
        for (int w = 1; w < T / 64; ++w) t = mode == LQ_MAX ? fmax(t, wpart[w]) : t + wpart[w];
    return t;
}

template <bool ROOT>
__device__ inline double lq_norm(double acc, int mode, double q)
{
    if (ROOT) return pow(acc, 1.0 / q);
    return mode == LQ_TWO ? sqrt(acc) : acc;
}

// The norm: a part per workgroup, added up by every workgroup of the pass behind it (fixed thread -> element map and fixed
// reduction tree, so the norm is the same bits in every run).
// ONCE: see ONCE_FROM.
template <Power P, bool ONCE>
__global__ __launch_bounds__(256) void lq_norm_pass(const float* __restrict__ g, long long n, int mode, double q,
                                                    double* __restrict__ partial)
{
    __shared__ double wpart[4];
    __shared__ PowerTable power;
    const int tid = threadIdx.x;
    if constexpr (P == TABLE) {
        make_power_table<256>(power, q);
        __syncthreads();
    }
    double acc = 0.0;
    auto visit = [&](float x) { acc = lq_add<P>(acc, x, mode, q, power); };
    const bool vec = (((size_t)g) & 15) == 0;
    const long long n4 = vec ? n / 4 : 0;
    const long long stride = (long long)gridDim.x * 256;
    for (long long q0 = (long long)blockIdx.x * 256 + tid; q0 < n4; q0 += 4 * stride) {
        float4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long qq = q0 + u * stride;
            x[u] = qq >= n4 ? make_float4(0.f, 0.f, 0.f, 0.f) : ONCE ? load_once((const float4*)g + qq) : ((const float4*)g)[qq];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) { visit(x[u].x); visit(x[u].y); visit(x[u].z); visit(x[u].w); }
    }
    for (long long i = n4 * 4 + (long long)blockIdx.x * 256 + tid; i < n; i += stride) visit(g[i]);
    const double part = lq_block_reduce<256>(acc, mode, wpart);
    if (tid == 0) partial[blockIdx.x] = part;
}

// The whole l_q encoder for n <= LOCAL_MAX.
template <Power P>
__global__ __launch_bounds__(LOCAL_T) void lq_encode_local(const float* __restrict__ g, int n, int mode, double q,
                                                           unsigned long long stream_id, unsigned long long seed,
                                                           long long capacity, unsigned int* __restrict__ idx, float* p_out,
                                                           float* norm_out, long long* count_out, int* flags)
{
    __shared__ double wpart[LOCAL_T / 64];
    __shared__ double norm_sh;
    __shared__ PowerTable power;
    float x[LOCAL_PER];
    local_load(g, n, x);
    if constexpr (P == TABLE) {
        make_power_table<LOCAL_T>(power, q);
        __syncthreads();
    }
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < LOCAL_PER; ++e)
        if (e / 4 * LOCAL_T * 4 < n) acc = lq_add<P>(acc, x[e], mode, q, power);
    const double t = lq_block_reduce<LOCAL_T>(acc, mode, wpart);
    if (threadIdx.x == 0) {
        norm_sh = lq_norm<P != PLAIN>(t, mode, q);
        *norm_out = (float)norm_sh;
    }
    __syncthreads();
    local_message<true>(x, n, norm_sh > 0.0 ? 1.0 / norm_sh : 0.0, stream_id, seed, capacity, idx, nullptr, p_out, count_out, flags);
}

// The l_q encoder's pass over the gradient behind the norm: draws against the exact p, one group of segments per workgroup.
template <int STEPS, bool ROOT, bool ONCE>
__global__ __launch_bounds__(256) void lq_draw(const float* __restrict__ g, long long n, EwState* st, const double* __restrict__ partial,
                                               int parts, int mode, double q, float* norm_out, unsigned long long stream_id,
                                               unsigned long long seed, Segments sg)
{
    __shared__ unsigned int wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __shared__ double wpart[4], ratio_sh;
    double acc = 0.0;
    for (int k = tid; k < parts; k += 256) acc = mode == LQ_MAX ? fmax(acc, partial[k]) : acc + partial[k];
    acc = lq_block_reduce<256>(acc, mode, wpart);
    if (tid == 0) {
        const double norm = lq_norm<ROOT>(acc, mode, q);
        ratio_sh = norm > 0.0 ? 1.0 / norm : 0.0;                // p_i = min(1, |g_i| / |g|_q)
        if (blockIdx.x == 0) {
            st->ratio = ratio_sh;
            *norm_out = (float)norm;
        }
    }
    __syncthreads();
    const double ratio = ratio_sh;
    const int mine = sg.per_group / 4;
    const long long seg0 = (long long)blockIdx.x * sg.per_group + wave * mine;
    unsigned int total = 0u;                                     // wave-uniform
    for (long long seg = seg0; seg < min(seg0 + mine, sg.n_seg); ++seg) {
        const Slots sl = lq_slots(sg, seg);
        const unsigned int kept = draw_segment<STEPS, ONCE>(g, n, seg, stream_id, seed, ratio,
            [&](unsigned int pos, unsigned int off, float x, float) {
                if (pos < (unsigned int)sl.capacity) sl.word[pos] = (unsigned short)(off | (x < 0.0f ? FLAG_BIT : 0u));
            });
        if (lane == 0) sg.count[seg] = kept | (kept > (unsigned int)sl.capacity ? OVER : 0u);
        total += kept;
    }
    if (lane == 0) wsum[wave] = total;
    __syncthreads();
    if (tid == 0) sg.group_kept[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

struct EwLayout {
    EwState* st;
    double* lq_partial;           // [LQ_WGS] per-workgroup parts of |g|_q
    unsigned long long* own;      // [SAMPLE_WGS][NBUCKET / 2] sampled levels, see ew_sample
    Segments sg;
    int steps;                    // float4 steps per segment
    size_t bytes;
};

// limit: bytes that may be used, 0 for no limit (the records take what is left; a segment that finds too few slots is drawn
// again, see "records").
EwLayout ew_layout(void* base, int64_t n, size_t limit = 0)
{
    Carver carve(base);
    EwLayout l;
    // Short segments until there are enough of them to fill the chip several times over (8192 waves run at once), then
    // long ones: a segment costs its counts and a chain of loads in every later kernel whatever its length.
    l.steps = n < LONG_FROM ? 4 : 16;
    const int64_t seg = (int64_t)l.steps * STEP;
    l.sg.n_seg = (n + seg - 1) / seg;
    // A workgroup that writes the message adds up the counts of all groups before its own: about a thousand at most.
    l.sg.per_group = 4;
    while (l.sg.per_group < MAX_GROUP && (l.sg.n_seg + l.sg.per_group - 1) / l.sg.per_group > 1024) l.sg.per_group *= 2;
    l.sg.n_groups = (l.sg.n_seg + l.sg.per_group - 1) / l.sg.per_group;
    l.st = carve.take<EwState>(1);
    l.lq_partial = carve.take<double>(LQ_WGS);
    l.sg.count = carve.take<unsigned int>((size_t)l.sg.n_seg);
    l.sg.group_kept = carve.take<unsigned int>((size_t)l.sg.n_groups);
    l.sg.open_max = (unsigned)(n / 4096 + 512);                  // (twice of what is to be expected of a message of all elements)
    l.sg.open = carve.take<EwOpen>(l.sg.open_max);
    l.sg.tally = sampled_levels(l.steps) ? carve.take<Tally>(DRAW_WGS) : nullptr;
    l.own = sampled_levels(l.steps) ? carve.take<unsigned long long>(SAMPLE_WGS * NBUCKET / 2) : nullptr;
    l.sg.spins = SPIN_COUNTED;
    size_t step_bytes = STEP_BYTES;
    if (limit) step_bytes = std::min<size_t>(step_bytes, (limit - carve.off - 256) / ((size_t)l.sg.n_seg * l.steps) & ~(size_t)7);
    l.sg.slot_bytes = (int)(step_bytes * l.steps);
    l.sg.slots = carve.take<unsigned char>((size_t)l.sg.n_seg * l.sg.slot_bytes);
    l.bytes = carve.off;
    return l;
}

// The state of the search lives outside the shared workspace: its histograms and tickets are handed from call to call zeroed
// (the last kernel of a call clears what it used), which saves a clearing launch at the head of every call.
int search_state(atomo_ctx* ctx, hipStream_t stream, EwState** st)
{
    if (!ctx->ew_state) {
        ATOMO_HIP(ctx, hipMalloc(&ctx->ew_state, sizeof(EwState)));
        ATOMO_HIP(ctx, hipMemsetAsync(ctx->ew_state, 0, sizeof(EwState), stream));
    }
    *st = (EwState*)ctx->ew_state;
    return ATOMO_OK;
}

// Workgroups of level 0: none may visit 2^16 elements or more (field widths of the packed histogram word).  Each adds some hundred buckets
// that are not empty to the global histogram, one by one, which takes longer than to read 32,768 elements instead of 4,096 (one million
// elements on 245 workgroups 11.3 us, on 64 8.4; four million on 256 13.1, on 128 11.5); below 64 of them the chip is too empty for that
// (60,000 on 15 6.5, on 4 7.6).
int level0_workgroups(int64_t n)
{
    const int64_t few = std::min<int64_t>(256, std::max<int64_t>(64, n / 32768));
    return (int)std::max<int64_t>(std::min<int64_t>(few, (n + 4095) / 4096), (n + 49151) / 49152);
}

}  // namespace

size_t entrywise_workspace_bytes(int64_t n) { return ew_layout(nullptr, n).bytes; }

namespace {

// The encoder proper: every buffer it needs beyond the caller's lies in `l`.  The histograms in l.st must be zero on
// entry and are zero again when the last kernel has run (clear_first: do not rely on that, clear them first).
int enqueue_encode_entrywise(atomo_ctx* ctx, const float* g, double s, uint64_t seed, uint64_t stream_id,
                             const atomo_ew_msg* msg, float* p_out, const EwLayout& l, bool clear_first, hipStream_t stream)
{
    const int64_t n = msg->n;
    if (n <= LOCAL_MAX) {
        ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream);
        ew_encode_local<<<1, LOCAL_T, 0, stream>>>(g, (int)n, s, stream_id, seed, (long long)msg->capacity, msg->idx, msg->val,
                                                   p_out, (long long*)msg->count, ctx->d_flags);
        ATOMO_HIP(ctx, hipGetLastError());
        return ATOMO_OK;
    }
    Segments sg = l.sg;
    if (ctx->ew_spins >= 0) sg.spins = ctx->ew_spins;
    const int wgs0 = level0_workgroups(n);
    const unsigned quads = (unsigned)((sg.n_seg + 3) / 4), groups = (unsigned)sg.n_groups;
    const bool long_seg = l.steps == 16;
    if (clear_first) { ProfScope ps(ctx, ATOMO_K_EW_SOLVE, stream); ew_clear<<<(3 * NBUCKET + 255) / 256, 256, 0, stream>>>(l.st); }
    if (long_seg) {
        const unsigned draws = std::min<unsigned>(quads, DRAW_WGS);
        { ProfScope ps(ctx, ATOMO_K_EW_HIST, stream); ew_sample<<<SAMPLE_WGS, 1024, 0, stream>>>(g, n, l.st, s, l.own); }
        { ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream); ew_draw<16, SAMPLED><<<draws, 256, 0, stream>>>(g, n, l.st, s, stream_id, seed, sg); }
        { ProfScope ps(ctx, ATOMO_K_EW_HIST, stream); ew_confirm<<<CONFIRM_WGS, 1024, 0, stream>>>(g, n, l.st, s, sg.tally, draws, (unsigned)align_up(wgs0, CONFIRM_WGS)); }
        { ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream); ew_draw<16, REDO><<<std::min<unsigned>(draws, REDO_WGS), 256, 0, stream>>>(g, n, l.st, s, stream_id, seed, sg); }
    } else {
        { ProfScope ps(ctx, ATOMO_K_EW_HIST, stream); ew_hist0_solve0<<<wgs0, 1024, 0, stream>>>(g, n, l.st, s); }
        { ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream); ew_draw<4, EXACT><<<quads, 256, 0, stream>>>(g, n, l.st, s, stream_id, seed, sg); }
    }
    {
        ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream);
        if (long_seg) ew_settle<16><<<groups, 256, 0, stream>>>(g, n, l.st, s, stream_id, seed, sg);
        else ew_settle<4><<<groups, 256, 0, stream>>>(g, n, l.st, s, stream_id, seed, sg);
        const auto write = long_seg ? ew_write<16, false> : ew_write<4, false>;
        write<<<groups, 256, 0, stream>>>(g, n, l.st, s, stream_id, seed, sg, (long long)msg->capacity, msg->idx, msg->val,
                                          (long long*)msg->count, ctx->d_flags);
        if (p_out) ew_write_p<<<(int)std::min<int64_t>(4096, (n + 255) / 256), 256, 0, stream>>>(g, n, l.st, p_out);
    }
    ATOMO_HIP(ctx, hipGetLastError());
    return ATOMO_OK;
}

}  // namespace

int encode_entrywise(atomo_ctx* ctx, const float* g, double s, uint64_t seed, uint64_t stream_id,
                     const atomo_ew_msg* msg, float* p_out, hipStream_t stream)
{
    const int64_t n = msg->n;
    int rc = ensure_workspace(ctx, entrywise_workspace_bytes(n));
    if (rc != ATOMO_OK) return rc;
    EwLayout l = ew_layout(ctx->ws, n);
    rc = search_state(ctx, stream, &l.st);
    if (rc != ATOMO_OK) return rc;
    return enqueue_encode_entrywise(ctx, g, s, seed, stream_id, msg, p_out, l, false, stream);
}

int encode_lq(atomo_ctx* ctx, const float* g, double q, uint64_t seed, uint64_t stream_id, const atomo_lq_msg* msg,
              float* p_out, hipStream_t stream)
{
    const int64_t n = msg->n;
    int rc = ensure_workspace(ctx, entrywise_workspace_bytes(n));
    if (rc != ATOMO_OK) return rc;
    EwLayout l = ew_layout(ctx->ws, n);
    rc = search_state(ctx, stream, &l.st);
    if (rc != ATOMO_OK) return rc;
    const int mode = std::isinf(q) ? LQ_MAX : q == 2.0 ? LQ_TWO : q == 1.0 ? LQ_ONE : LQ_POW;
    // (not for one element per thread: the table takes a pow per thread itself, whether there is something to raise or not; 300 elements 7.4 us by
    // the table, 7.5 without, one in 200 of them not zero 7.3 and 6.0; 2000 elements 7.6 and 8.6)
    const bool table = q <= TABLE_Q && n > LOCAL_T;
    if (n <= LOCAL_MAX) {
        ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream);
        const auto encode = mode != LQ_POW ? lq_encode_local<PLAIN> : table ? lq_encode_local<TABLE> : lq_encode_local<POW>;
        encode<<<1, LOCAL_T, 0, stream>>>(g, (int)n, mode, q, stream_id, seed, (long long)msg->capacity, msg->idx, p_out,
                                                   msg->norm, (long long*)msg->count, ctx->d_flags);
        ATOMO_HIP(ctx, hipGetLastError());
        return ATOMO_OK;
    }
    const int wgs = (int)std::min<int64_t>(LQ_WGS, (n + 4095) / 4096);
    const bool once = n >= ONCE_FROM;
    static_assert(ONCE_FROM >= LONG_FROM, "segments of 16 steps");
    {
        ProfScope ps(ctx, ATOMO_K_EW_HIST, stream);              // the norm pass takes the place of the histograms
        const auto pass = once ? (mode != LQ_POW ? lq_norm_pass<PLAIN, true> : table ? lq_norm_pass<TABLE, true> : lq_norm_pass<POW, true>)
                               : (mode != LQ_POW ? lq_norm_pass<PLAIN, false> : table ? lq_norm_pass<TABLE, false> : lq_norm_pass<POW, false>);
        pass<<<wgs, 256, 0, stream>>>(g, n, mode, q, l.lq_partial);
    }
    {
        ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream);
        const unsigned groups = (unsigned)l.sg.n_groups;
        const bool long_seg = l.steps == 16;
        const auto draw = once ? (mode == LQ_POW ? lq_draw<16, true, true> : lq_draw<16, false, true>)
                        : long_seg ? (mode == LQ_POW ? lq_draw<16, true, false> : lq_draw<16, false, false>)
                                   : (mode == LQ_POW ? lq_draw<4, true, false> : lq_draw<4, false, false>);
        draw<<<groups, 256, 0, stream>>>(g, n, l.st, l.lq_partial, wgs, mode, q, msg->norm, stream_id, seed, l.sg);
        const auto write = long_seg ? ew_write<16, true> : ew_write<4, true>;
        write<<<groups, 256, 0, stream>>>(g, n, l.st, 0.0, stream_id, seed, l.sg, (long long)msg->capacity, msg->idx, nullptr,
                                          (long long*)msg->count, ctx->d_flags);
        if (p_out) ew_write_p<<<(int)std::min<int64_t>(4096, (n + 255) / 256), 256, 0, stream>>>(g, n, l.st, p_out);
    }
    ATOMO_HIP(ctx, hipGetLastError());
    return ATOMO_OK;
}

int probabilities(atomo_ctx* ctx, const float* lambda, const int64_t* offsets, int n_seg, double s, float* p,
                  hipStream_t stream)
{
    std::vector<char>& table = ctx->table_scratch;
    table.clear();
    std::vector<int> large;
    int n_local = 0;
    for (int k = 0; k < n_seg; ++k) {
        const int64_t len = offsets[k + 1] - offsets[k];
        if (len == 0) continue;
        if (len <= LOCAL_MAX) {
            const LocalSeg seg{(long long)offsets[k], (int)len, 0};
            table.insert(table.end(), (const char*)&seg, (const char*)(&seg + 1));
            ++n_local;
        } else {
            large.push_back(k);
        }
    }
    void* d_segs = nullptr;
    if (n_local) {
        const int rc = resident_tables(ctx, ctx->prob_tables, table, stream, &d_segs);
        if (rc != ATOMO_OK) return rc;
    }
    EwState* st = nullptr;
    if (!large.empty()) {
        const int rc = search_state(ctx, stream, &st);
        if (rc != ATOMO_OK) return rc;
    }
    for (size_t j = 0; j < std::max<size_t>(large.size(), n_local ? 1 : 0); ++j) {
        const bool any = j < large.size();
        const int64_t begin = any ? offsets[large[j]] : 0, len = any ? offsets[large[j] + 1] - begin : 0;
        const float* x = lambda + begin;
        const int beside = j == 0 ? n_local : 0;                 // the short segments ride along with the first long one
        prob_first<<<(unsigned)(beside + (any ? level0_workgroups(len) : 0)), LOCAL_T, 0, stream>>>(
            lambda, (const LocalSeg*)d_segs, beside, s, p, x, len, st);
        if (!any) break;
        const int wgs = (int)std::max<int64_t>(std::min<int64_t>(HIST_WGS, (len + 4095) / 4096), (len + 49151) / 49152);
        ew_hist<1><<<wgs, 256, 0, stream>>>(x, len, st, s);
        ew_hist<2><<<wgs, 256, 0, stream>>>(x, len, st, s);
        prob_last<<<(int)std::min<int64_t>(1024, (len + 1023) / 1024), 256, 0, stream>>>(x, len, st, s, p + begin);
    }
    ATOMO_HIP(ctx, hipGetLastError());
    return ATOMO_OK;
}

}  // namespace atomo

// ---------------------------------------------------------------------------------------------------------
// atomo_encode_entrywise_noalloc: the entry-wise encoder for callers that cannot allocate (see include/atomo.h).
// Its scratch memory (the state of the water-level search, counts and records) is the
// file-scope device array below instead of the context's growable workspace.  Every GPU the library runs on
// holds its own copy of the array, at its own address, until the process ends; the address on a device is
// looked up once, with that device current (atomo_create does it, so that no call made later has to).
// ---------------------------------------------------------------------------------------------------------
namespace {

constexpr long long NOALLOC_MAX_N = 1ll << 24;                   // 16,777,216 elements (64 MiB of gradient)
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)5 << 20;        // 5 MiB per GPU
constexpr int NOALLOC_MAX_DEVICES = 64;

static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

// Device address of `scratch` per HIP device (the array's name is only a host-side handle for the symbol).
void* scratch_ptr[NOALLOC_MAX_DEVICES];

}  // namespace

namespace atomo {

// Called with ctx->device current.  Looks the address up on the first call for a device.
int entrywise_noalloc_setup(atomo_ctx* ctx)
{
    const int dev = ctx->device;
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return ATOMO_EINVAL;
    if (__atomic_load_n(&scratch_ptr[dev], __ATOMIC_ACQUIRE)) return ATOMO_OK;
    if (ew_layout(nullptr, NOALLOC_MAX_N, NOALLOC_SCRATCH_BYTES).bytes > NOALLOC_SCRATCH_BYTES) return ATOMO_EINVAL;   // (a build-time fact)
    void* ptr = nullptr;
    ATOMO_HIP(ctx, hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return ATOMO_EHIP;
    __atomic_store_n(&scratch_ptr[dev], ptr, __ATOMIC_RELEASE);   // (two threads racing here store the same address)
    return ATOMO_OK;
}

}  // namespace atomo

extern "C" int atomo_encode_entrywise_noalloc(atomo_ctx* ctx, const float* g, double s, uint64_t seed, uint64_t stream_id,
                                              const atomo_ew_msg* msg, float* p_out, void* stream)
{
    using namespace atomo;
    if (!ctx || !g || !msg || !(s > 0.0) || std::isinf(s)) return ATOMO_EINVAL;
    if (msg->n <= 0 || msg->capacity < 1 || !msg->count || !msg->idx || !msg->val) return ATOMO_EINVAL;
    if (msg->n > NOALLOC_MAX_N) return ATOMO_ETOOLARGE;
    int prev = -1;
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != ctx->device) ATOMO_HIP(ctx, hipSetDevice(ctx->device));
    int rc = entrywise_noalloc_setup(ctx);                        // a table look-up after atomo_create
    if (rc == ATOMO_OK) {
        // event bracketing of launches creates events on demand: not on this path
        const bool profiling = ctx->profiling;
        ctx->profiling = false;
        void* base = __atomic_load_n(&scratch_ptr[ctx->device], __ATOMIC_ACQUIRE);
        // (the array keeps what the previous call left: the histograms are cleared first, by a kernel)
        rc = enqueue_encode_entrywise(ctx, g, s, seed, stream_id, msg, p_out, ew_layout(base, msg->n, NOALLOC_SCRATCH_BYTES), true, (hipStream_t)stream);
        ctx->profiling = profiling;
    }
    if (prev >= 0 && prev != ctx->device) (void)hipSetDevice(prev);
    return rc;
}

