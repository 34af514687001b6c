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
// draw every uniform against the bracket that level 0 leaves for p_i.  Whatever may be kept is written down in that pass as
// a record (value and offset), and all that follows reads the records, a hundredth of the gradient: the third level of the
// search, the settling of the few draws inside the bracket, the message.  The l_q encoder (Section 4), whose probabilities
// need only a norm, draws against the exact p and has nothing to settle.
#include <cmath>
#include <vector>

#include "atomo_internal.h"
#include "block_algorithm1.h"

namespace atomo {

namespace {

constexpr int L0_BITS = 11, L1_BITS = 10, L2_BITS = 10;
constexpr int NBUCKET = 1 << L0_BITS;        // the largest level
constexpr int HIST_WGS = 1024;

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
};

struct EwState {
    unsigned int cnt[3][NBUCKET];
    unsigned long long sig[3][NBUCKET];
    SolveOut lvl[3];              // what each level found (written by one kernel, read by the kernels after it);
                                  // lvl[k].done also when an earlier level already settled everything
    unsigned int ticket[3][65];   // per pass: workgroups that have finished (the last one solves the level); zero between calls
    unsigned long long n_s;       // final: number of capped elements
    double tail;                  // final: sum of the uncapped magnitudes
    double budget;                // final: s - n_s
    double ratio;                 // final: budget / tail, +inf if tail == 0
    unsigned long long total_kept;
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

__global__ __launch_bounds__(256) void ew_clear(EwState* st)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < 3 * NBUCKET) { (&st->cnt[0][0])[i] = 0u; (&st->sig[0][0])[i] = 0ull; }
    if (i == 0) {
        for (int k = 0; k < 3 * 65; ++k) (&st->ticket[0][0])[k] = 0u;
        for (int k = 0; k < 3; ++k) { st->lvl[k].done = 0; st->lvl[k].prefix = 0u; st->lvl[k].n_above = 0ull; st->lvl[k].sum_below = 0.0; }
        st->n_s = 0ull; st->tail = 0.0; st->budget = 0.0; st->ratio = 0.0; st->total_kept = 0ull;
    }
}

// Level-LEVEL histogram of the elements on the path `prefix`, by the TPB threads of a workgroup (all call):
// accumulated in the LDS array acc (COPIES x NB packed words), then added to the global histogram.
template <int LEVEL, int TPB>
__device__ inline void hist_body(const float* __restrict__ g, long long n, EwState* st, unsigned long long* acc, unsigned int prefix)
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
    const long long n4 = vec ? n / 4 : 0;
    const long long stride = (long long)gridDim.x * TPB;
    // four loads in flight per thread: one at a time, the pass is a chain of memory latencies
    for (long long q0 = (long long)blockIdx.x * TPB + threadIdx.x; q0 < n4; q0 += 4 * stride) {
        float4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long q = q0 + u * stride;
            if (q < n4) x[u] = ((const float4*)g)[q];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (q0 + u * stride < n4) { visit(x[u].x); visit(x[u].y); visit(x[u].z); visit(x[u].w); }
        }
    }
    for (long long i = n4 * 4 + (long long)blockIdx.x * TPB + threadIdx.x; i < n; i += stride) visit(g[i]);
    __syncthreads();
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

// Histogram of one level.  Elements are visited as float4 where the pointer allows.
template <int LEVEL>
__global__ __launch_bounds__(LEVEL == 0 ? 1024 : 256) void ew_hist(const float* __restrict__ g, long long n, EwState* st)
{
    constexpr int TPB = LEVEL == 0 ? 1024 : 256;
    __shared__ unsigned long long acc[(LEVEL == 0 ? 4 : 1) * (LEVEL == 0 ? (1 << L0_BITS) : (1 << L1_BITS))];
    if (LEVEL > 0 && st->lvl[LEVEL > 0 ? LEVEL - 1 : 0].done) return;
    hist_body<LEVEL, TPB>(g, n, st, acc, LEVEL == 0 ? 0u : st->lvl[LEVEL > 0 ? LEVEL - 1 : 0].prefix);
}

// One level of the search, by the T threads of a workgroup (all must call).
// Reads the level's histogram from st, and the path chosen so far from `in` (level 0: nothing).  The result goes
// to `out` (LDS or global, visible to the workgroup after the call's last barrier).
// T threads (256 or 1024); COHERENT: the histogram was written by other workgroups of the running kernel (atomics), so it
// is read with device-scope atomic loads instead of plain ones.
// scratch: LDS, (2 T / 64 + 1) x 8 bytes.
template <int LEVEL, int T = 256, bool COHERENT = false>
__device__ inline void solve_level(const EwState* st, double s, unsigned int prefix, unsigned long long n_above0,
                                   double sum_below0, SolveOut* out, unsigned long long* scratch)
{
    unsigned long long* cpart = scratch;
    double* spart = (double*)(scratch + T / 64);
    int& best = *(int*)(scratch + 2 * (T / 64));
    constexpr int NB = LEVEL == 0 ? (1 << L0_BITS) : (1 << L1_BITS);
    constexpr int SHIFT = LEVEL == 0 ? 20 : LEVEL == 1 ? 10 : 0;
    constexpr int PER = NB / T;
    static_assert(PER >= 1, "one bucket per thread at least");
    const int tid = threadIdx.x;
    auto bucket_key = [&](int b) -> unsigned int {
        return ((LEVEL == 0 ? 0u : prefix << (LEVEL == 1 ? L1_BITS : L2_BITS)) | (unsigned int)b) << SHIFT;
    };
    // exponent shared by every element on the chosen path (level 0: part of the bucket index)
    auto bucket_exp = [&](int b) -> unsigned int { return bucket_key(b) >> 23; };
    auto bucket_lo = [&](int b) -> double { return (double)__uint_as_float(bucket_key(b)); };

    // this thread's PER consecutive buckets stay in registers
    unsigned int cnt_r[PER];
    double sum_r[PER];
    unsigned long long c_mine = 0ull;
    double s_mine = 0.0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int b = tid * PER + e;
        if (COHERENT) {                                          // (both loads in flight at once)
            cnt_r[e] = __hip_atomic_load(&st->cnt[LEVEL][b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long sg = __hip_atomic_load(&st->sig[LEVEL][b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sum_r[e] = cnt_r[e] ? sig_value(sg, bucket_exp(b)) : 0.0;
        } else {
            cnt_r[e] = st->cnt[LEVEL][b];
            sum_r[e] = cnt_r[e] ? sig_value(st->sig[LEVEL][b], bucket_exp(b)) : 0.0;    // (most buckets are empty)
        }
        c_mine += cnt_r[e];
        s_mine += sum_r[e];
    }
    __syncthreads();                                             // (the scratch may still be read from a previous call)
    // suffix scan of the counts and prefix scan of the sums over the threads: in the wave by shuffles, then over the waves
    const int lane = tid & 63, wave = tid >> 6;
    unsigned long long c_scan = c_mine;
    double s_scan = s_mine;
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long cv = __shfl_down(c_scan, off);
        const double sv = __shfl_up(s_scan, off);
        if (lane + off < 64) c_scan += cv;
        if (lane >= off) s_scan += sv;
    }
    if (lane == 0) cpart[wave] = c_scan;
    if (lane == 63) spart[wave] = s_scan;
    if (tid == 0) best = 0;
    __syncthreads();
    unsigned long long c_after = c_scan - c_mine;                // count in buckets owned by later threads
    double s_before = __shfl_up(s_scan, 1);                      // sum in buckets owned by earlier threads
    if (lane == 0) s_before = 0.0;
    {
        double earlier = 0.0;
        for (int w = 0; w < T / 64; ++w) {
            if (w > wave) c_after += cpart[w];
            if (w < wave) earlier += spart[w];
        }
        s_before += earlier;
    }

    // h at the lower edge of bucket b:  lo_b * (s - #{elements in buckets >= b}) - sum(buckets < b)
    {
        unsigned long long at_or_above = c_after + c_mine;
        double below = s_before;
        int mine_best = -1;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int b = tid * PER + e;
            const double h = bucket_lo(b) * (s - (double)(n_above0 + at_or_above)) - (sum_below0 + below);
            if (h <= 0.0) mine_best = b;
            at_or_above -= cnt_r[e];
            below += sum_r[e];
        }
        if (mine_best >= 0) atomicMax(&best, mine_best);
    }
    __syncthreads();
    const int bs = best;
    if (tid == bs / PER) {                      // the owner of the chosen bucket finishes from its registers
        unsigned long long above = c_after;
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
        out->n_s = n_s;
        out->tail = tail;
        out->n_above = n_above;
        out->sum_below = sum_below;
        out->prefix = (LEVEL == 0 ? 0u : prefix << (LEVEL == 1 ? L1_BITS : L2_BITS)) | (unsigned int)bs;
        out->lo = bucket_lo(bs);
        out->hi = bs + 1 < NB ? bucket_lo(bs + 1) : __longlong_as_double(0x7FF0000000000000LL);
    }
    __syncthreads();
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

template <int LEVEL>
__global__ __launch_bounds__(256) void ew_solve(EwState* st, double s)
{
    __shared__ SolveOut out;
    __shared__ unsigned long long scratch[2 * 4 + 1];
    unsigned int prefix = 0u;
    unsigned long long n_above = 0ull;
    double sum_below = 0.0;
    if (LEVEL > 0) {
        const SolveOut& in = st->lvl[LEVEL > 0 ? LEVEL - 1 : 0];
        if (in.done) {                                           // settled earlier: hand the mark on
            if (threadIdx.x == 0) st->lvl[LEVEL].done = 1;
            return;
        }
        prefix = in.prefix; n_above = in.n_above; sum_below = in.sum_below;
    }
    solve_level<LEVEL>(st, s, prefix, n_above, sum_below, &out, scratch);
    if (threadIdx.x == 0) publish(st, LEVEL, out, s);
}

// True in every thread of the workgroup that finishes last among the launch's workgroups (all threads of every
// workgroup call, at their very end).  The last workgroup may then read what the others added to the global
// histograms, with device-scope atomic loads: every wave first waits until its own atomics have been performed
// (s_waitcnt vmcnt(0): on gfx9 stores and atomics count in vmcnt, and a workgroup barrier alone does not wait for memory
// operations in flight), and device-scope atomics are performed where every compute unit sees them, so no cache
// maintenance is involved.  Nobody waits for anybody: the others simply leave.
// Tickets in two levels (thousands of atomic adds on one address are performed one after the other, about ten
// nanoseconds each): a workgroup counts on word blockIdx.x mod 64, the last one of a word counts on word 64.
// ticket: [65] words, zero on entry and zero again when the last workgroup returns.
__device__ inline bool last_workgroup(unsigned int* ticket)
{
    __shared__ int last_sh;
    __builtin_amdgcn_s_waitcnt(0x0F70);                          // vmcnt(0), other counters untouched
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned int slots = min(64u, gridDim.x), slot = blockIdx.x % slots;
        const unsigned int members = (gridDim.x - slot + slots - 1) / slots;
        int last = 0;
        if (__hip_atomic_fetch_add(&ticket[slot], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == members - 1)
            last = __hip_atomic_fetch_add(&ticket[64], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == slots - 1;
        last_sh = last;
    }
    __syncthreads();
    if (last_sh && threadIdx.x < 65)                             // for the next call
        __hip_atomic_store(&ticket[threadIdx.x], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return last_sh != 0;
}

// ew_hist<0> whose last workgroup solves level 0 at once: one launch and one chain of dependent loads less than with
// ew_solve<0> behind it.
__global__ __launch_bounds__(1024) void ew_hist0_solve0(const float* __restrict__ g, long long n, EwState* st, double s)
{
    __shared__ unsigned long long acc[4 * NBUCKET];
    __shared__ SolveOut out;
    hist_body<0, 1024>(g, n, st, acc, 0u);
    if (!last_workgroup(st->ticket[0])) return;
    solve_level<0, 1024, true>(st, s, 0u, 0ull, 0.0, &out, acc);            // (acc is spent: scratch)
    if (threadIdx.x == 0) publish(st, 0, out, s);
}

// p = min(1, |x| (s - n_s) / tail) (eq. (p_i), KKT appendix); `ratio` = (s - n_s) / tail in double,
// or +inf when nothing is left uncapped.  One double multiply and one rounding to float per element.
__device__ inline float ew_probability(float x, double ratio)
{
    const float a = fabsf(x);
    if (a == 0.0f) return 0.0f;
    return fminf(1.0f, (float)((double)a * ratio));
}

// p for a large segment of atomo_probabilities
__global__ __launch_bounds__(256) void ew_write_p(const float* __restrict__ lam, long long n, const EwState* st,
                                                  float* __restrict__ p)
{
    const double ratio = st->ratio;
    const long long stride = (long long)gridDim.x * 256;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += stride)
        p[i] = ew_probability(lam[i], ratio);
}

// Draws for the four coordinates 4q .. 4q+3 (one Philox block).  Returns the keep bits.
__device__ inline unsigned int draw4(const float4 x, long long q, unsigned long long stream_id, unsigned long long seed,
                                     double ratio, float4& p)
{
    const u32x4 rnd = philox4x32_10((unsigned long long)q, stream_id, seed);
    p.x = ew_probability(x.x, ratio);
    p.y = ew_probability(x.y, ratio);
    p.z = ew_probability(x.z, ratio);
    p.w = ew_probability(x.w, ratio);
    return (u01(rnd.x) < p.x ? 1u : 0u) | (u01(rnd.y) < p.y ? 2u : 0u) | (u01(rnd.z) < p.z ? 4u : 0u) |
           (u01(rnd.w) < p.w ? 8u : 0u);
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
constexpr unsigned int DIRECT_MAX = 65536;

struct Segments {
    unsigned int* count;          // [n_seg] records of a segment; in a group with an OVER among them: kept coordinates | OVER
    unsigned int* group_kept;     // [n_groups] kept coordinates of a group of per_group segments
    unsigned char* slots;
    long long n_seg, n_groups;
    int slot_bytes;               // per segment
    int per_group;
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

// Calls visit(position, offset in the segment, value, p) for every kept coordinate of a segment, drawn from the gradient
// with the exact ratio; returns their number.  All lanes of the wave call.
template <int STEPS, typename VISIT>
__device__ inline unsigned int draw_segment(const float* __restrict__ g, long long n, long long seg,
                                            unsigned long long stream_id, unsigned long long seed, double ratio, VISIT visit)
{
    const bool vec = (((size_t)g) & 15) == 0;
    const int lane = threadIdx.x & 63;
    unsigned int fill = 0u;                                      // wave-uniform
    for (int j = 0; j < STEPS; ++j) {
        const long long q = (seg * STEPS + j) * 64 + lane;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f), p = x;
        unsigned int bits = 0u;
        if (q * 4 < n) {
            x = load4(g, q, n, vec);
            bits = draw4(x, q, stream_id, seed, ratio, p);
        }
        unsigned long long ballots[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) ballots[e] = __ballot((bits >> e) & 1u);
        unsigned int pos = fill + listed_before(ballots);
        const float xs[4] = {x.x, x.y, x.z, x.w}, ps[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if ((bits >> e) & 1u) visit(pos++, (unsigned int)(j * STEP + lane * 4 + e), xs[e], ps[e]);
        fill += listed_total(ballots);
    }
    return fill;
}

// Second pass of the entry-wise encoder over the gradient; the level-0 result is read from st->lvl[0] (the launch before
// left it there).
// After level 0 the water level tau = tail / (s - n_s) is known to lie inside one bucket [lo, hi] of the float bit pattern
// (12.5 % wide), so p_i = min(1, |g_i| / tau) is bracketed for every element, and because rounding is monotone,
// fl(|g_i| / hi) <= p_i <= fl(|g_i| / lo)  holds for the float32 p_i that the final ratio will give.  An element is dropped
// here if u >= p_hi, marked as kept for sure if u < p_lo; what lies between (about 0.12 s elements) is settled by ew_settle
// once the remaining levels have fixed tau exactly.  Every element of the chosen bucket has p_hi >= 1 and so a record: level
// 1 is histogrammed here and level 2 from the records.
// Bound by the Philox rounds (18 wide multiplications per four elements): everything per element that can be left to the
// candidates, one element in fifty, is left to them.  2^28 elements, 1 % kept: 264 us, where drawing, keep bits, and gathering
// the kept values from the gradient again took 388 + 103 + 141 us and level 2, which read the gradient too, 202 us (now: 264,
// 22 for level 2, 21 to settle, 19 to write).
template <int STEPS>
__global__ __launch_bounds__(256) void ew_draw(const float* __restrict__ g, long long n, EwState* st, double s,
                                               unsigned long long stream_id, unsigned long long seed, Segments sg)
{
    __shared__ unsigned int l1cnt[1 << L1_BITS];
    __shared__ unsigned long long l1sig[1 << L1_BITS];
    const int tid = threadIdx.x, lane = tid & 63;
    const long long seg = (long long)blockIdx.x * 4 + (tid >> 6);
    const SolveOut so = st->lvl[0];
    const bool done = so.done != 0;
    const double inf = __longlong_as_double(0x7FF0000000000000LL);
    // Single-precision brackets of the p that the final ratio will give, p = fl32(|g| ratio), scaled by 2^24 like the
    // uniform (an integer below 2^24): with r_lo <= ratio (1 - 2^-22) and r_hi >= ratio (1 + 2^-22),
    // fl32(|g| r_lo) (1 - 2^-22) <= p <= fl32(|g| r_hi) (each rounding moves a value by at most 2^-24 of itself; where
    // |g| r_hi 2^24 underflows, p is zero).  A bracket that is a little wide only sends a few more coordinates to ew_settle,
    // which decides with the exact formula.
    double ratio_lo, ratio_hi;
    if (done) {
        ratio_lo = ratio_hi = final_ratio(s, so.n_s, so.tail);
    } else {
        ratio_lo = so.hi < inf ? 1.0 / so.hi : 0.0;              // 1 / hi <= ratio <= 1 / lo
        ratio_hi = so.lo > 0.0 ? 1.0 / so.lo : inf;
    }
    const double down = 1.0 - 4.76837158203125e-07, up = 1.0 + 4.76837158203125e-07;     // 1 -+ 2^-21, of the ratios
    // a ratio beyond the float range is bounded from below by the largest float and from above by infinity
    const float r_lo = ratio_lo < 1.0e31 ? (float)(ratio_lo * 16777216.0 * down) : 3.0e38f;
    const float r_hi = ratio_hi < 1.0e31 ? (float)(ratio_hi * 16777216.0 * up) : __int_as_float(0x7f800000);
    const bool zeros = !(ratio_hi < 1.0e31);                     // 0 * infinity: zeros are taken out by hand
    const unsigned int bucket = done ? 0xFFFFFFFFu : so.prefix;
    // Few elements in the bucket: straight into the global histogram, where they hardly ever meet.  Many: through LDS.
    const bool through_lds = !done && so.count > DIRECT_MAX;
    if (through_lds) {
        for (int b = tid; b < (1 << L1_BITS); b += 256) { l1cnt[b] = 0u; l1sig[b] = 0ull; }
        __syncthreads();
    }

    if (seg < sg.n_seg) {
        const bool vec = (((size_t)g) & 15) == 0;
        const Slots sl = ew_slots(sg, seg);
        unsigned int fill = 0u;                                  // wave-uniform
        for (int j0 = 0; j0 < STEPS; j0 += 4) {
            float4 xv[4];
            const long long q0 = (seg * STEPS + j0) * 64 + lane;
#pragma unroll
            for (int u = 0; u < 4; ++u) xv[u] = load4(g, q0 + u * 64, n, vec);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const u32x4 rnd = philox4x32_10((unsigned long long)(unsigned int)(q0 + u * 64), stream_id, seed);
                const float xs[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
                const float us[4] = {(float)(rnd.x >> 8), (float)(rnd.y >> 8), (float)(rnd.z >> 8), (float)(rnd.w >> 8)};
                bool in[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) in[e] = !(us[e] >= fabsf(xs[e]) * r_hi);     // (a NaN is a candidate)
                if (zeros) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) in[e] = in[e] && xs[e] != 0.0f;
                }
                unsigned long long ballots[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) ballots[e] = __ballot(in[e]);
                if (ballots[0] | ballots[1] | ballots[2] | ballots[3]) {
                    unsigned int pos = fill + listed_before(ballots);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (in[e]) {
                            const bool sure = us[e] < fminf(16777216.0f, fabsf(xs[e]) * r_lo) * (1.0f - 2.384185791015625e-07f);
                            if (pos < (unsigned int)sl.capacity) {
                                sl.val[pos] = xs[e];
                                sl.word[pos] = (unsigned short)(((j0 + u) * STEP + lane * 4 + e) | (sure ? FLAG_BIT : 0u));
                            }
                            ++pos;
                            const unsigned int key = __float_as_uint(xs[e]) & 0x7FFFFFFFu;
                            if ((key >> 20) == bucket) {
                                const unsigned int b = (key >> 10) & ((1 << L1_BITS) - 1);
                                if (through_lds) {
                                    atomicAdd(&l1cnt[b], 1u);
                                    atomicAdd(&l1sig[b], (unsigned long long)significand(key));
                                } else {
                                    atomicAdd(&st->cnt[1][b], 1u);
                                    atomicAdd(&st->sig[1][b], (unsigned long long)significand(key));
                                }
                            }
                        }
                    }
                    fill += listed_total(ballots);
                }
            }
        }
        if (lane == 0) sg.count[seg] = fill <= (unsigned int)sl.capacity ? fill : OVER;
    }
    if (done) {
        if (blockIdx.x == 0 && tid == 0) st->lvl[1].done = 1;    // nothing left for the levels below
        return;
    }
    if (through_lds) {
        __syncthreads();
        for (int b = tid; b < (1 << L1_BITS); b += 256) {
            const unsigned int cnt = l1cnt[b];
            if (cnt) {
                atomicAdd(&st->cnt[1][b], cnt);
                atomicAdd(&st->sig[1][b], l1sig[b]);
            }
        }
    }
    // the last workgroup to finish solves level 1 from the merged histogram
    if (!last_workgroup(st->ticket[1])) return;
    __shared__ SolveOut out;
    solve_level<1, 256, true>(st, s, so.prefix, so.n_above, so.sum_below, &out, l1sig);     // (l1sig is spent: scratch)
    if (tid == 0) publish(st, 1, out, s);
}

// Level-2 histogram of the elements on the path that level 1 chose, from the records (nothing to do if level 1 settled
// everything); its last workgroup solves level 2.
template <int STEPS>
__global__ __launch_bounds__(256) void ew_level2(const float* __restrict__ g, long long n, EwState* st, double s, Segments sg)
{
    __shared__ unsigned int cnt[1 << L2_BITS];
    __shared__ unsigned long long sig[1 << L2_BITS];
    __shared__ Group gr;
    __shared__ SolveOut out;
    const SolveOut in = st->lvl[1];
    if (in.done) return;
    const int tid = threadIdx.x;
    for (int b = tid; b < (1 << L2_BITS); b += 256) { cnt[b] = 0u; sig[b] = 0ull; }
    auto visit = [&](float x) {
        const unsigned int key = __float_as_uint(x) & 0x7FFFFFFFu;
        if ((key >> L2_BITS) == in.prefix) {
            atomicAdd(&cnt[key & ((1 << L2_BITS) - 1)], 1u);
            atomicAdd(&sig[key & ((1 << L2_BITS) - 1)], (unsigned long long)significand(key));
        }
    };
    for (long long group = blockIdx.x; group < sg.n_groups; group += gridDim.x) {
        load_group(sg, group, gr);
        __syncthreads();
        if (gr.over) {
            const long long i0 = group * sg.per_group * STEPS * STEP;
            const long long i1 = min(n, i0 + (long long)sg.per_group * STEPS * STEP);
            for (long long i = i0 + tid; i < i1; i += 256) visit(g[i]);
        } else {
            for (unsigned int t = tid; t < gr.before[MAX_GROUP]; t += 256) {
                const int k = segment_of(gr, sg.per_group, t);
                visit(ew_slots(sg, group * sg.per_group + k).val[t - gr.before[k]]);
            }
        }
        __syncthreads();
    }
    for (int b = tid; b < (1 << L2_BITS); b += 256) {
        if (cnt[b]) {
            atomicAdd(&st->cnt[2][b], cnt[b]);
            atomicAdd(&st->sig[2][b], sig[b]);
        }
    }
    if (!last_workgroup(st->ticket[2])) return;
    solve_level<2, 256, true>(st, s, in.prefix, in.n_above, in.sum_below, &out, sig);
    if (tid == 0) publish(st, 2, out, s);
}

// Settles the records of a group of segments with the final ratio: the draw of an open one is repeated, and what is not kept
// is marked.  Leaves the kept count of the group.
template <int STEPS>
__global__ __launch_bounds__(256) void ew_settle(const float* __restrict__ g, long long n, const EwState* st,
                                                 unsigned long long stream_id, unsigned long long seed, Segments sg)
{
    __shared__ unsigned int wsum[4];
    __shared__ Group gr;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double ratio = st->ratio;                              // final since the last solve
    const long long first = (long long)blockIdx.x * sg.per_group;
    load_group(sg, blockIdx.x, gr);
    __syncthreads();
    unsigned int kept = 0u;                                      // wave-uniform
    if (gr.over) {
        for (int k = wave; k < sg.per_group && first + k < sg.n_seg; k += 4) {
            const unsigned int c = draw_segment<STEPS>(g, n, first + k, stream_id, seed, ratio,
                                                       [](unsigned int, unsigned int, float, float) {});
            if (lane == 0) sg.count[first + k] = c | OVER;
            kept += c;
        }
    } else {
        for (unsigned int t0 = 0; t0 < gr.before[MAX_GROUP]; t0 += 256) {
            const unsigned int t = t0 + tid;
            bool keep = false;
            if (t < gr.before[MAX_GROUP]) {
                const int k = segment_of(gr, sg.per_group, t);
                const Slots sl = ew_slots(sg, first + k);
                const unsigned int r = t - gr.before[k], word = sl.word[r];
                const float x = sl.val[r];
                keep = (word & FLAG_BIT) != 0u;
                if (!keep) {
                    const unsigned int off = word & (FLAG_BIT - 1);
                    const u32x4 rnd = philox4x32_10((unsigned long long)((first + k) * STEPS * 64 + (off >> 2)), stream_id, seed);
                    const unsigned int bits = (off & 2) ? ((off & 1) ? rnd.w : rnd.z) : ((off & 1) ? rnd.y : rnd.x);
                    keep = u01(bits) < ew_probability(x, ratio);
                    if (!keep) sl.word[r] = (unsigned short)(word | DROPPED);
                }
            }
            kept += (unsigned int)__popcll(__ballot(keep));
        }
    }
    if (lane == 0) wsum[wave] = kept;
    __syncthreads();
    if (tid == 0) sg.group_kept[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// The message from the settled records, one group of segments per workgroup, which adds up the counts of all groups before
// its own by itself.  The last group also reports the total.
// LQ: every record is kept, and the message's words are index and sign (bit 31) alone.
template <int STEPS, bool LQ>
__global__ __launch_bounds__(256) void ew_write(const float* __restrict__ g, long long n, EwState* st,
                                                unsigned long long stream_id, unsigned long long seed, Segments sg,
                                                long long capacity, unsigned int* __restrict__ idx, float* __restrict__ val,
                                                long long* count_out, int* flags)
{
    __shared__ unsigned long long bsum[4];
    __shared__ unsigned int wsum[2][4];
    __shared__ Group gr;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double ratio = st->ratio;
    const long long first = (long long)blockIdx.x * sg.per_group;
    unsigned long long part = 0ull;
    for (long long i = tid; i < (long long)blockIdx.x; i += 256) part += sg.group_kept[i];
    load_group(sg, blockIdx.x, gr);
    for (int o = 32; o > 0; o >>= 1) part += __shfl_down(part, o);
    if (lane == 0) bsum[wave] = part;
    __syncthreads();
    unsigned long long base = bsum[0] + bsum[1] + bsum[2] + bsum[3];
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
            const unsigned long long pos0 = base + gr.before[k];
            const unsigned int i0 = (unsigned int)((first + k) * STEPS * STEP);
            draw_segment<STEPS>(g, n, first + k, stream_id, seed, ratio,
                                [&](unsigned int pos, unsigned int off, float x, float p) { put(pos0 + pos, i0 + off, x, p); });
        }
        base += gr.before[MAX_GROUP];
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
        st->total_kept = base;
        *count_out = (long long)base;
        if ((long long)base > capacity) atomicMax(&flags[FLAG_CAPACITY], 1);
    }
    if (!LQ) {   // the histograms have had their last reader: zero again for the next call
        for (long long i = (long long)blockIdx.x * 256 + tid; i < 3 * NBUCKET; i += (long long)gridDim.x * 256) {
            (&st->cnt[0][0])[i] = 0u;
            (&st->sig[0][0])[i] = 0ull;
        }
    }
}

// Small segments of atomo_probabilities: sort-based Algorithm 1, one workgroup per segment.
struct SmallSeg { long long begin; int n; int pad; };

__global__ __launch_bounds__(256) void prob_small(const float* __restrict__ lam, const SmallSeg* segs, double s,
                                                  float* __restrict__ p)
{
    __shared__ float key[ALG1_MAX];
    __shared__ int src[ALG1_MAX];
    __shared__ Alg1Scratch sc;
    const SmallSeg seg = segs[blockIdx.x];
    const int n = seg.n, tid = threadIdx.x;
    if (n <= 0) return;
    int P = 1;
    while (P < n) P <<= 1;
    for (int i = tid; i < P; i += 256) {
        key[i] = i < n ? fabsf(lam[seg.begin + i]) : -1.0f;
        src[i] = i;
    }
    __syncthreads();
    block_sort_desc(key, src, P);
    const int ns = block_algorithm1(key, n, s, sc);
    const double tail_ns = sc.tail_ns;
    for (int i = tid; i < n; i += 256) p[seg.begin + src[i]] = alg1_probability(key[i], i, ns, s, tail_ns);
}

// ---- l_q quantisation (Section 4) -------------------------------------------------------------------
enum { LQ_MAX = 0, LQ_TWO = 1, LQ_ONE = 2, LQ_POW = 3 };
constexpr int LQ_WGS = 1024;

// Per-workgroup part of |g|_q: max |g_i|, or the sum of g_i^2, |g_i| or |g_i|^q in double (fixed thread ->
// element map and fixed reduction tree, so the norm is the same bits in every run).
__global__ __launch_bounds__(256) void lq_norm_partial(const float* __restrict__ g, long long n, int mode, double q,
                                                       double* __restrict__ partial)
{
    __shared__ double wpart[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double acc = 0.0;
    auto visit = [&](float x) {
        const double a = (double)fabsf(x);
        if (mode == LQ_MAX) acc = fmax(acc, a);
        else if (mode == LQ_TWO) acc = fma(a, a, acc);
        else if (mode == LQ_ONE) acc += a;
        else if (a > 0.0) acc += pow(a, q);
    };
    const bool vec = (((size_t)g) & 15) == 0;
    const long long n4 = vec ? n / 4 : 0;
    const long long stride = (long long)gridDim.x * 256;
    for (long long q0 = (long long)blockIdx.x * 256 + tid; q0 < n4; q0 += 4 * stride) {
        float4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long qq = q0 + u * stride;
            x[u] = qq < n4 ? ((const float4*)g)[qq] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) { visit(x[u].x); visit(x[u].y); visit(x[u].z); visit(x[u].w); }
    }
    for (long long i = n4 * 4 + (long long)blockIdx.x * 256 + tid; i < n; i += stride) visit(g[i]);
    for (int o = 32; o > 0; o >>= 1) {
        const double other = __shfl_down(acc, o);
        acc = mode == LQ_MAX ? fmax(acc, other) : acc + other;
    }
    if (lane == 0) wpart[wave] = acc;
    __syncthreads();
    if (tid == 0) {
        double t = wpart[0];
        for (int w = 1; w < 4; ++w) t = mode == LQ_MAX ? fmax(t, wpart[w]) : t + wpart[w];
        partial[blockIdx.x] = t;
    }
}

// |g|_q from the partial results (one workgroup), 1 / |g|_q as the sampler's ratio, and the message's norm.
__global__ __launch_bounds__(256) void lq_norm_final(const double* __restrict__ partial, int n_partial, int mode, double q,
                                                     EwState* st, float* norm_out)
{
    __shared__ double tree[256];
    const int tid = threadIdx.x;
    double t = 0.0;
    for (int k = tid; k < n_partial; k += 256) t = mode == LQ_MAX ? fmax(t, partial[k]) : t + partial[k];
    tree[tid] = t;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (tid < off) tree[tid] = mode == LQ_MAX ? fmax(tree[tid], tree[tid + off]) : tree[tid] + tree[tid + off];
        __syncthreads();
    }
    if (tid == 0) {
        const double acc = tree[0];
        const double norm = mode == LQ_MAX || mode == LQ_ONE ? acc : mode == LQ_TWO ? sqrt(acc) : pow(acc, 1.0 / q);
        st->ratio = norm > 0.0 ? 1.0 / norm : 0.0;               // p_i = min(1, |g_i| / |g|_q)
        st->n_s = 0ull; st->tail = norm; st->budget = 1.0; st->total_kept = 0ull;
        for (int k = 0; k < 3; ++k) st->lvl[k].done = 1;
        *norm_out = (float)norm;
    }
}

// The l_q encoder's pass over the gradient behind the norm: draws against the exact p, one group of segments per workgroup.
template <int STEPS>
__global__ __launch_bounds__(256) void lq_draw(const float* __restrict__ g, long long n, const EwState* st,
                                               unsigned long long stream_id, unsigned long long seed, Segments sg)
{
    __shared__ unsigned int wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double ratio = st->ratio;
    const int mine = sg.per_group / 4;
    const long long seg0 = (long long)blockIdx.x * sg.per_group + wave * mine;
    unsigned int total = 0u;                                     // wave-uniform
    for (long long seg = seg0; seg < min(seg0 + mine, sg.n_seg); ++seg) {
        const Slots sl = lq_slots(sg, seg);
        const unsigned int kept = draw_segment<STEPS>(g, n, seg, stream_id, seed, ratio,
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
    l.steps = n < (1ll << 25) ? 4 : 16;
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
    size_t step_bytes = STEP_BYTES;
    if (limit) step_bytes = std::min<size_t>(step_bytes, (limit - carve.off - 256) / ((size_t)l.sg.n_seg * l.steps) & ~(size_t)7);
    l.sg.slot_bytes = (int)(step_bytes * l.steps);
    l.sg.slots = carve.take<unsigned char>((size_t)l.sg.n_seg * l.sg.slot_bytes);
    l.bytes = carve.off;
    return l;
}

// Enqueues the three histogram / solve levels; afterwards st->{n_s, tail, budget} are final.
void enqueue_water_level(atomo_ctx* ctx, const float* x, int64_t n, double s, EwState* st, hipStream_t stream)
{
    // No workgroup may visit 2^16 elements or more (field widths of the packed histogram word).
    const int64_t floor_wgs = (n + 49151) / 49152;
    const int wgs = (int)std::max<int64_t>(std::min<int64_t>(HIST_WGS, (n + 1023) / 1024), floor_wgs);
    const int wgs0 = (int)std::max<int64_t>(std::min<int64_t>(256, (n + 4095) / 4096), floor_wgs);
    { ProfScope ps(ctx, ATOMO_K_EW_SOLVE, stream); ew_clear<<<(3 * NBUCKET + 255) / 256, 256, 0, stream>>>(st); }
    { ProfScope ps(ctx, ATOMO_K_EW_HIST, stream); ew_hist<0><<<wgs0, 1024, 0, stream>>>(x, n, st); }
    { ProfScope ps(ctx, ATOMO_K_EW_SOLVE, stream); ew_solve<0><<<1, 256, 0, stream>>>(st, s); }
    { ProfScope ps(ctx, ATOMO_K_EW_HIST, stream); ew_hist<1><<<wgs, 256, 0, stream>>>(x, n, st); }
    { ProfScope ps(ctx, ATOMO_K_EW_SOLVE, stream); ew_solve<1><<<1, 256, 0, stream>>>(st, s); }
    { ProfScope ps(ctx, ATOMO_K_EW_HIST, stream); ew_hist<2><<<wgs, 256, 0, stream>>>(x, n, st); }
    { ProfScope ps(ctx, ATOMO_K_EW_SOLVE, stream); ew_solve<2><<<1, 256, 0, stream>>>(st, s); }
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
    const Segments& sg = l.sg;
    // No workgroup may visit 2^16 elements or more (field widths of the packed histogram word).
    const int64_t floor_wgs = (n + 49151) / 49152;
    const int wgs0 = (int)std::max<int64_t>(std::min<int64_t>(256, (n + 4095) / 4096), floor_wgs);
    const int wgs2 = (int)std::min<int64_t>(HIST_WGS, sg.n_groups);
    const unsigned quads = (unsigned)((sg.n_seg + 3) / 4), groups = (unsigned)sg.n_groups;
    const bool long_seg = l.steps == 16;
    if (clear_first) { ProfScope ps(ctx, ATOMO_K_EW_SOLVE, stream); ew_clear<<<(3 * NBUCKET + 255) / 256, 256, 0, stream>>>(l.st); }
    { ProfScope ps(ctx, ATOMO_K_EW_HIST, stream); ew_hist0_solve0<<<wgs0, 1024, 0, stream>>>(g, n, l.st, s); }
    {
        ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream);
        if (long_seg) ew_draw<16><<<quads, 256, 0, stream>>>(g, n, l.st, s, stream_id, seed, sg);
        else ew_draw<4><<<quads, 256, 0, stream>>>(g, n, l.st, s, stream_id, seed, sg);
    }
    {
        ProfScope ps(ctx, ATOMO_K_EW_HIST, stream);
        if (long_seg) ew_level2<16><<<wgs2, 256, 0, stream>>>(g, n, l.st, s, sg);
        else ew_level2<4><<<wgs2, 256, 0, stream>>>(g, n, l.st, s, sg);
    }
    {
        ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream);
        if (long_seg) ew_settle<16><<<groups, 256, 0, stream>>>(g, n, l.st, stream_id, seed, sg);
        else ew_settle<4><<<groups, 256, 0, stream>>>(g, n, l.st, stream_id, seed, sg);
        const auto write = long_seg ? ew_write<16, false> : ew_write<4, false>;
        write<<<groups, 256, 0, stream>>>(g, n, l.st, stream_id, seed, sg, (long long)msg->capacity, msg->idx, msg->val,
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
    // The search state lives outside the shared workspace: its histograms are handed from call to call zeroed (the
    // last kernel of a call clears them), which saves the clearing launch at the head of every call.
    if (!ctx->ew_state) {
        ATOMO_HIP(ctx, hipMalloc(&ctx->ew_state, sizeof(EwState)));
        ATOMO_HIP(ctx, hipMemsetAsync(ctx->ew_state, 0, sizeof(EwState), stream));
    }
    EwLayout l = ew_layout(ctx->ws, n);
    l.st = (EwState*)ctx->ew_state;
    return enqueue_encode_entrywise(ctx, g, s, seed, stream_id, msg, p_out, l, false, stream);
}

int encode_lq(atomo_ctx* ctx, const float* g, double q, uint64_t seed, uint64_t stream_id, const atomo_lq_msg* msg,
              float* p_out, hipStream_t stream)
{
    const int64_t n = msg->n;
    int rc = ensure_workspace(ctx, entrywise_workspace_bytes(n));
    if (rc != ATOMO_OK) return rc;
    const EwLayout l = ew_layout(ctx->ws, n);
    const int mode = std::isinf(q) ? LQ_MAX : q == 2.0 ? LQ_TWO : q == 1.0 ? LQ_ONE : LQ_POW;
    const int wgs = (int)std::min<int64_t>(LQ_WGS, (n + 4095) / 4096);
    {
        ProfScope ps(ctx, ATOMO_K_EW_HIST, stream);              // the norm pass takes the place of the histograms
        lq_norm_partial<<<wgs, 256, 0, stream>>>(g, n, mode, q, l.lq_partial);
    }
    { ProfScope ps(ctx, ATOMO_K_EW_SOLVE, stream); lq_norm_final<<<1, 256, 0, stream>>>(l.lq_partial, wgs, mode, q, l.st, msg->norm); }
    {
        ProfScope ps(ctx, ATOMO_K_EW_SAMPLE, stream);
        const unsigned groups = (unsigned)l.sg.n_groups;
        const bool long_seg = l.steps == 16;
        if (long_seg) lq_draw<16><<<groups, 256, 0, stream>>>(g, n, l.st, stream_id, seed, l.sg);
        else lq_draw<4><<<groups, 256, 0, stream>>>(g, n, l.st, stream_id, seed, l.sg);
        const auto write = long_seg ? ew_write<16, true> : ew_write<4, true>;
        write<<<groups, 256, 0, stream>>>(g, n, l.st, stream_id, seed, l.sg, (long long)msg->capacity, msg->idx, nullptr,
                                          (long long*)msg->count, ctx->d_flags);
        if (p_out) ew_write_p<<<(int)std::min<int64_t>(4096, (n + 255) / 256), 256, 0, stream>>>(g, n, l.st, p_out);
    }
    ATOMO_HIP(ctx, hipGetLastError());
    return ATOMO_OK;
}

int probabilities(atomo_ctx* ctx, const float* lambda, const int64_t* offsets, int n_seg, double s, float* p,
                  hipStream_t stream)
{
    std::vector<SmallSeg> small;
    std::vector<int> large;
    for (int k = 0; k < n_seg; ++k) {
        const int64_t len = offsets[k + 1] - offsets[k];
        if (len == 0) continue;
        if (len <= ALG1_MAX) small.push_back(SmallSeg{(long long)offsets[k], (int)len, 0});
        else large.push_back(k);
    }
    size_t need = align_up(small.size() * sizeof(SmallSeg), 256) + 256;
    if (!large.empty()) need += align_up(sizeof(EwState), 256);
    int rc = ensure_workspace(ctx, need);
    if (rc != ATOMO_OK) return rc;
    Carver carve(ctx->ws);
    SmallSeg* d_small = carve.take<SmallSeg>(small.size());
    EwState* st = large.empty() ? nullptr : carve.take<EwState>(1);
    if (!small.empty()) {
        rc = upload(ctx, d_small, small.data(), small.size() * sizeof(SmallSeg), stream);
        if (rc != ATOMO_OK) return rc;
        prob_small<<<(unsigned)small.size(), 256, 0, stream>>>(lambda, d_small, s, p);
    }
    for (int k : large) {
        const int64_t len = offsets[k + 1] - offsets[k];
        const float* x = lambda + offsets[k];
        enqueue_water_level(ctx, x, len, s, st, stream);
        const int wgs = (int)std::min<int64_t>(4096, (len + 255) / 256);
        ew_write_p<<<wgs, 256, 0, stream>>>(x, len, st, p + offsets[k]);
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

