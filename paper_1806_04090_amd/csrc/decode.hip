// Decoders (eq. (vhat) of arXiv 1806.04090): g_hat = sum over kept atoms of (lambda_i / p_i) a_i.
//
// SVD messages: out = scale * sum_msgs sum_k w_k u_k v_k^T, a dense rank-(sum k) update written once.
// Each workgroup owns a 64 x 256 tile of one output and contracts the atoms of every message summed into
// it on the matrix cores.  Few atoms (one worker, budget 3): bound by the HBM write of the tile.  Many
// (the average over 16 workers, rank ~ 48): the 2 m n K flops take as long on the fp32 matrix cores as the write,
// and the workgroups, which all start together, go through listing, products and stores in step.
// The same kernel adds the update to what `out` holds instead of overwriting it (the parameter server's step,
// params += alpha * average gradient), and takes messages in the folded form (weight inside U).
// Entry-wise and l_q messages: one launch that searches the messages' ascending coordinates (decode_sparse).
#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

#include "atomo_internal.h"
#include "svd_device.h"

namespace atomo {

namespace {

struct DecMsg {
    const int* count;
    const float* w;
    const float* U;
    const float* V;
    int capacity;
    int pad;
};

struct DecOut {
    float* out;
    long long ld;
    int rows, cols;
    int first, last;           // messages [first, last)
};

struct DecWork { int out, tile_r, tile_c, pad; };

constexpr int TR = 64, TC = 256;
constexpr int TALL_ROWS = 256;     // rows per workgroup for outputs of at most 32 columns
constexpr int ATOMS_MAX = 512;     // atoms listed in LDS at a time

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// out tile (64 x 256) = sum over messages and kept atoms of (scale w_k u_k) v_k^T as a rank-K update on the
// matrix cores: A operand (row i, atom k) = scale w_k U[k][i], B operand (atom k, column j) = V[k][j],
// v_mfma_f32_32x32x2f32, two atoms per instruction.  Wave w owns columns 64 w .. 64 w + 63 of the tile as
// 2 x 2 blocks of 32 x 32.
// The kept atoms of a batch of messages (`batch` x largest capacity <= ATOMS_MAX, chosen by the host) are first
// listed in LDS: by one wave, a message per lane, its place from a scan over the counts in registers, or, where it is
// one message, by all threads (a thread per message that added the counts before its own up in LDS, a barrier more
// and a second trip for the message behind it: the 131072 x 18 and the other layers of Section 6 23.5 us, now 17.5;
// the update from 8 27.4, now 26.5).  The operands then come through LDS in pieces of KP atoms: all
// 256 threads fetch the piece's slices of u (64 rows) and v (256 columns) with 16-byte loads that are all in
// flight at once - every atom's u and v are contiguous rows of its message -, and the loads of the next piece
// are issued before the products of the current one.  The weight is applied on the way into LDS.
// A message with a capacity above ATOMS_MAX is a batch of its own and is listed and contracted in runs of
// ATOMS_MAX atoms.
// TALL: outputs of at most 32 columns (the [x*y/2, 2*k*k] reshape of Section 6).  The workgroup owns 256 rows,
// wave w rows 64 w .. 64 w + 63, one 32-column block.
constexpr int KP = 16;             // atoms per piece (8 and 24 measure the same; 32 leaves room for two workgroups per
                                   // compute unit instead of four and is a third slower)

// sum over the lanes of the wave up to this one
__device__ inline int inclusive_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast 15 to rows 1 and 3, 31 to rows 2 and 3
    return x + __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
}

struct DecLds {
    Global<const float> up[ATOMS_MAX];
    Global<const float> vp[ATOMS_MAX];
    Global<const float> wp[ATOMS_MAX];                           // the atom's weight (nullptr: folded into u)
    int total, span;
    __attribute__((aligned(16))) float operands[KP * (TR + TC + 64)];
};

template <bool TALL, bool ACCUMULATE>
__device__ __forceinline__ void decode_tile(DecLds& lds, const DecOut* outs, const DecMsg* msgs, const DecWork* work, float scale, int batch)
{
    constexpr int NCB = TALL ? 1 : 2;
    constexpr int UROWS = TALL ? TALL_ROWS : TR;                 // rows of the tile = length of a u slice
    constexpr int VCOLS = TALL ? 32 : TC;                        // columns of the tile = length of a v slice
    constexpr int US = UROWS + 32, VS = VCOLS + 32;              // LDS strides: odd and even atoms on different banks
    constexpr int NU = (KP * UROWS / 4 + 255) / 256;             // 16-byte loads per thread and piece, u and v
    constexpr int NV = (KP * VCOLS / 4 + 255) / 256;
    static_assert(US + VS <= TR + TC + 64, "operands in the LDS of either form");
    Global<const float> *const up = lds.up, *const vp = lds.vp, *const wp = lds.wp;
    float *const Us = lds.operands, *const Vs = lds.operands + KP * US;
    const DecWork wk = work[blockIdx.x];
    const DecOut o = outs[wk.out];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, l32 = lane & 31;
    const int tile_r0 = TALL ? wk.tile_r * TALL_ROWS : wk.tile_r * TR;
    const int tile_c0 = TALL ? 0 : wk.tile_c * TC;
    const int row_off = TALL ? wave * 64 : 0, col_off = TALL ? 0 : wave * 64;    // this wave's corner inside the tile
    floatx16 acc[2][NCB];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[rb][cb][v] = 0.0f;

    // this lane's corner; element v of block (rb, cb): row below(rb, v) under it, column 32 cb to its right
    const int row0 = tile_r0 + row_off + 4 * h, col0 = tile_c0 + col_off + l32;
    auto below = [](int rb, int v) { return rb * 32 + 8 * (v >> 2) + (v & 3); };
    // the tile as it is, on its way from here on: 36.9 -> 28.1 us for the update of 9.75 M parameters from 8 messages (a load
    // behind each store of the end waits for it)
    floatx16 old[2][NCB];
    if constexpr (ACCUMULATE) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                const Global<const float> in = global((const float*)o.out) + min(col0 + cb * 32, o.cols - 1);
#pragma unroll
                for (int v = 0; v < 16; ++v) old[rb][cb][v] = in[(long long)min(row0 + below(rb, v), o.rows - 1) * o.ld];
            }
    }

    // four consecutive elements of an atom's row, zero beyond `limit`; one 16-byte load where the address allows
    auto load4 = [](Global<const float> base, int at, int limit) {
        float4 x = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        const Global<const float> p = base + at;
        if (at + 3 < limit && (((size_t)p) & 15) == 0) {
            const floatx4 y = *(Global<const floatx4>)p;
            x = make_float4(y[0], y[1], y[2], y[3]);
        } else {
            if (at < limit) x.x = p[0];
            if (at + 1 < limit) x.y = p[1];
            if (at + 2 < limit) x.z = p[2];
            if (at + 3 < limit) x.w = p[3];
        }
        return x;
    };
    float4 ru[NU], rv[NV];
    float rw[NU];
    // the loads of the piece that starts at list position k0 (positions from `total` on read as zero).  Nothing is done with
    // them here: a product with the weight would wait for them in front of the products that they are to run beside
    // (16 workers' ResNet-18 24.9 -> 23.8 us, the update of VGG-11-BN from 8 29.6 -> 27.9)
    auto fetch = [&](int k0, int total) {
#pragma unroll
        for (int e = 0; e < NU; ++e) {
            const int f = tid + 256 * e, atom = f / (UROWS / 4), part = f % (UROWS / 4);
            ru[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            rw[e] = 1.0f;
            if (atom < KP && k0 + atom < total) {
                const Global<const float> w = wp[k0 + atom];
                if (w) rw[e] = *w;
                ru[e] = load4(up[k0 + atom], tile_r0 + 4 * part, o.rows);
            }
        }
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            const int f = tid + 256 * e, atom = f / (VCOLS / 4), part = f % (VCOLS / 4);
            rv[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (atom < KP && k0 + atom < total) rv[e] = load4(vp[k0 + atom], tile_c0 + 4 * part, o.cols);
        }
    };
    // the first `here` atoms of the piece are there; the others are zero whatever the scale is (infinity times a padding of zeros
    // would be NaN, in every element of the tile)
    auto stage = [&](int here) {
#pragma unroll
        for (int e = 0; e < NU; ++e) {
            const int f = tid + 256 * e, atom = f / (UROWS / 4), part = f % (UROWS / 4);
            const float w = atom < here ? scale * rw[e] : 0.0f;
            if (atom < KP) *(float4*)&Us[atom * US + 4 * part] = make_float4(w * ru[e].x, w * ru[e].y, w * ru[e].z, w * ru[e].w);
        }
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            const int f = tid + 256 * e, atom = f / (VCOLS / 4), part = f % (VCOLS / 4);
            if (atom < KP) *(float4*)&Vs[atom * VS + 4 * part] = rv[e];
        }
    };

    // atoms [run, run + ATOMS_MAX) of the messages [first, first + nm) (several have no more than that together, by the host's choice
    // of `batch`; one alone is taken in runs)
    auto list = [&](int first, int nm, int run) {
        auto put = [&](const DecMsg& m, int at, int k) {
            up[at] = global(m.U) + (size_t)k * o.rows;
            vp[at] = global(m.V) + (size_t)k * o.cols;
            wp[at] = m.w ? global(m.w) + k : nullptr;            // folded messages carry the weight in U
        };
        if (nm == 1) {
            const DecMsg m = msgs[first];
            const int kept = min(*global(m.count), m.capacity), here = max(0, min(kept - run, ATOMS_MAX));
            int mine = tid;
            // (or the addresses below are worked out once in front of all batches, and six registers of every lane kept in scratch
            // memory: 46.6 MiB written for the 42.6 of ResNet-18, 22.6 us for 16 workers, now 22.2.  The other form has registers left)
            if (!ACCUMULATE) asm volatile("" : "+v"(mine));
            for (int k = mine; k < here; k += 256) put(m, k, run + k);
            if (tid == 0) {
                lds.total = here;
                lds.span = kept;
            }
        } else if (wave == 0) {
            int before = 0;
            for (int q0 = 0; q0 < nm; q0 += 64) {                // (one round trip for all counts)
                const bool there = q0 + lane < nm;
                const DecMsg m = msgs[first + min(q0 + lane, nm - 1)];
                const int kept = there ? min(*global(m.count), m.capacity) : 0;
                const int upto = before + inclusive_sum(kept);
                for (int k = 0, at = upto - kept; k < kept && at < ATOMS_MAX; ++k, ++at) put(m, at, k);
                before = __builtin_amdgcn_readlane(upto, 63);
            }
            if (lane == 0) {
                lds.total = min(before, ATOMS_MAX);
                lds.span = 0;
            }
        }
    };

    auto products = [&](int here) {
        const int pairs = (min(KP, here) + 1) / 2;
        for (int t = 0; t < pairs; ++t) {
            const float* ua = &Us[(2 * t + h) * US + row_off + l32];
            const float* vb = &Vs[(2 * t + h) * VS + col_off + l32];
            const float a0 = ua[0], a1 = ua[32], b0 = vb[0];
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);
            if (!TALL) {
                const float b1 = vb[32];
                acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
                acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);
            }
        }
    };
    for (int first = o.first; first < o.last; first += batch) {
        const int nm = min(batch, o.last - first);
        for (int run = 0, span = 1; run < span; run += ATOMS_MAX) {
            if (run > 0 || first > o.first) __syncthreads();     // the previous list is spent
            list(first, nm, run);
            __syncthreads();
            span = lds.span;
            const int total = lds.total;
            if (total > 0) fetch(0, total);
            for (int k0 = 0; k0 < total; k0 += KP) {
                stage(total - k0);
                __syncthreads();
                if (k0 + KP < total) fetch(k0 + KP, total);
                products(total - k0);
                __syncthreads();                                 // the piece is spent
            }
        }
    }
    // A narrow tile without gaps is one piece of memory: through LDS, and out in rows of 16 bytes per lane, where a row of the products is 18
    // lanes of 32 (the layers of ResNet-18 in the Section 6 reshape, 11.16 M outputs: 17.9 -> 16.5 us; with several tiles one after the
    // other in a workgroup, and one list of atoms for them, 24)
    if constexpr (TALL && !ACCUMULATE) {
        if (o.ld == o.cols && o.cols * TALL_ROWS <= KP * (TR + TC + 64)) {
            const int cols = o.cols;
            if (l32 < cols) {
#pragma unroll
                for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                    for (int v = 0; v < 16; ++v) lds.operands[(row_off + 4 * h + below(rb, v)) * cols + l32] = acc[rb][0][v];
            }
            __syncthreads();
            const int here = min(TALL_ROWS, o.rows - tile_r0) * cols;
            const Global<float> to = global(o.out) + (long long)tile_r0 * cols;
            const int quads = (((size_t)to) & 15) == 0 ? here / 4 : 0;
            for (int k = tid; k < quads; k += 256) *(Global<floatx4>)(to + 4 * k) = *(const floatx4*)&lds.operands[4 * k];
            for (int k = 4 * quads + tid; k < here; k += 256) to[k] = lds.operands[k];
            return;
        }
    }
    const Global<float> corner = global(o.out) + (long long)row0 * o.ld + col0;
    // A whole tall tile: no look at the row in front of every store, which is a branch each (600,000 rows, three atoms of each of four
    // messages: 25 columns 24.8 -> 21.9 us, 24 columns with gaps 26.3 -> 23.0; 23.2 and 24.9 without the form above beside them)
    if constexpr (TALL && !ACCUMULATE) {
        if (tile_r0 + TALL_ROWS <= o.rows) {
            if (l32 < o.cols) {
#pragma unroll
                for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                    for (int v = 0; v < 16; ++v) corner[below(rb, v) * o.ld] = acc[rb][0][v];
            }
            return;
        }
    }
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (row0 + below(rb, v) < o.rows && col0 + cb * 32 < o.cols)
                    corner[below(rb, v) * o.ld + cb * 32] = ACCUMULATE ? old[rb][cb][v] + acc[rb][cb][v] : acc[rb][cb][v];
}

// The first n_wide items of `work` are 64 x 256 tiles, the others (TALL: there are some) tall ones; both in one launch, or a few of one
// kind are a launch that nothing runs beside (the layers of ResNet-18 in the Section 6 reshape 22.3 -> 18.0 us).
// (128 registers for four workgroups per compute unit; with the outputs in registers too, 63 of them would go to memory for three)
template <bool TALL, bool ACCUMULATE>
__global__ __launch_bounds__(256, ACCUMULATE ? 1 : 4) void decode_svd_tiles(const DecOut* outs, const DecMsg* msgs, const DecWork* work,
                                                        int n_wide, float scale, int batch)
{
    __shared__ DecLds lds;
    if (!TALL || (int)blockIdx.x < n_wide) decode_tile<false, ACCUMULATE>(lds, outs, msgs, work, scale, batch);
    else decode_tile<true, ACCUMULATE>(lds, outs, msgs, work, scale, batch);
}

// ------------------------------------------------------------------------------------------------
// Entry-wise and l_q messages.  The kept coordinates of a message ascend, so a workgroup that owns SPARSE_TILE
// consecutive outputs finds its own part of every message by a search, adds the parts up in LDS in the order of
// the messages and writes its outputs once: one launch for a fill and a scatter per message, and the outputs of
// several messages are not read back.  Inside a message the coordinates are distinct, so plain LDS read-add-writes
// with a barrier between messages give the same bits in every run.
// Bound: HBM write of the outputs.  11.17 M outputs, one message of 111,740 pairs: 14.1 us, 11.4 without LDS
// (decode_sparse_one; 8.6 us a fill + 4.1 us a scatter, as two launches); 16 messages 34 us (8.6 + 16 x 4.1); 268 M outputs 228 us (187 + 110).
// The descriptors travel in the kernel's arguments (SPARSE_MSGS of them: half a kilobyte), nothing is uploaded.
// ------------------------------------------------------------------------------------------------
constexpr int SPARSE_TILE = 4096;      // outputs per workgroup: 16 KB of LDS, eight workgroups per compute unit
constexpr int SPARSE_RESIDENT = 2048;  // workgroups the chip holds at once
constexpr int SPARSE_MSGS = 16;        // messages per launch
constexpr int64_t ONE_ANY = 1 << 22;   // outputs, and tiles, up to which one message decodes without LDS (see the dispatch)
constexpr int ONE_TILES = 8192;
// Outputs from here on (384 MB) go around the last cache, which could not hold them: what is written into it drives out what others wrote,
// and the pass behind this one waits for the rest (2^28 outputs 230 -> 207 us and the search behind it 3 faster, 180 million 152 -> 140,
// 100 million 75 -> 72; 70 million 47 -> 52).  With an encode or an update behind the decode that holds for any message (150 million outputs,
// a ten-thousandth kept, encode and decode 250 -> 245, decode and update 426 -> 422); a decode alone, into the same buffer again, gains from
// three in a thousand on and loses 3 % below.
constexpr long long AROUND_FROM = 96'000'000;

struct SparseMsg {
    const long long* count;
    const unsigned int* idx;
    const float* val;          // entry-wise: [capacity] values; l_q: [1] the magnitude
    long long capacity;
};

struct SparseMsgs {
    SparseMsg m[SPARSE_MSGS];
    int n;
};

// First position in idx[0, kept) whose coordinate (masked) is not below `key`, by groups of G lanes of a wave, a search
// of its own per group: every round of loads narrows the range G + 1 times.
template <int G>
__device__ inline long long lower_bound_group(const unsigned int* idx, long long kept, unsigned int mask, unsigned int key)
{
    const int lane = threadIdx.x & 63, glane = lane & (G - 1), shift = lane & ~(G - 1);
    const unsigned long long members = G == 64 ? ~0ull : (1ull << (G & 63)) - 1;
    auto below = [&](long long at, bool valid) {                 // how many of the group's probes are below
        const bool b = valid && (idx[at] & mask) < key;
        return __popcll((__ballot(b) >> shift) & members);
    };
    long long lo = 0, len = kept;
    while (__any(len > G)) {                                     // (groups that are done repeat an empty round)
        const bool active = len > G;
        const long long step = (len + G) / (G + 1);              // G probes split the range into G + 1 pieces
        const long long at = lo + (glane + 1) * step - 1;
        const int c = below(at, active && at < lo + len);
        if (active) {
            lo += c * step;
            len -= c * step;
            if (c < G) len = min(step - 1, len);                 // (the probe at the end of the piece is not below)
        }
    }
    return lo + below(lo + glane, glane < len);
}

// Share `number` of `shares` of a message's pairs: do their coordinates ascend?
__device__ inline void check_order(const SparseMsg& m, int number, int shares, unsigned int mask, int* flags)
{
    const long long pairs = min(*m.count, m.capacity) - 1, share = (pairs + shares - 1) / shares;
    const long long from = number * share, to = min(pairs, from + share);
    bool disorder = false;
    for (long long k0 = from + threadIdx.x; k0 < to; k0 += 256 * 8) {    // sixteen loads in flight
        unsigned int a[8], b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const long long k = min(k0 + 256 * u, to - 1);
            a[u] = m.idx[k] & mask;
            b[u] = m.idx[k + 1] & mask;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) disorder |= a[u] >= b[u];
    }
    if (disorder) atomicMax(&flags[FLAG_ORDER], 1);
}

// One message: nothing is added up, so the outputs need not go through LDS.  Three waves write the zeros of the workgroup's tile,
// from the start and without waiting for anything, while the fourth searches; the values follow behind the barrier (stores of
// a workgroup to one place are performed in the order that the barrier gives them).  The searching wave has no stores of its own in
// front of its loads, which would be waited for first.
// Bound: the write of the outputs.  11.17 M outputs, 111,740 pairs: 14.1 -> 11.4 us (the stores waited for the search); one l_q
// message of 3343 pairs 11.2 -> 9.3.
template <bool LQ>
__global__ __launch_bounds__(256) void decode_sparse_one(SparseMsg m, float scale, float* __restrict__ out, long long n, int checks,
                                                         int* flags)
{
    __shared__ long long at_sh;
    const unsigned int mask = LQ ? 0x7FFFFFFFu : 0xFFFFFFFFu;
    if ((int)blockIdx.x < checks) {
        check_order(m, blockIdx.x, checks, mask, flags);
        return;
    }
    const int tid = threadIdx.x, wave = tid >> 6;
    const long long first = (long long)(blockIdx.x - checks) * SPARSE_TILE;
    const int here = (int)min(n - first, (long long)SPARSE_TILE);
    float* const o = out + first;
    const long long kept = min(*m.count, m.capacity);
    if (wave == 0) {
        const long long at = lower_bound_group<64>(m.idx, kept, mask, (unsigned int)first);
        if (tid == 0) at_sh = at;
    } else {
        const int quads = (((size_t)out) & 15) == 0 ? here / 4 : 0;
        for (int k = tid - 64; k < quads; k += 192) *(float4*)(o + 4 * k) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        for (int k = 4 * quads + tid - 64; k < here; k += 192) o[k] = 0.0f;
    }
    __syncthreads();
    const float mag = LQ ? scale * *m.val : 0.0f;
    for (long long k = at_sh + tid; k < kept; k += 256) {
        const unsigned int w = m.idx[k];
        const long long i = (long long)(w & mask) - first;
        if (i >= here) break;                                    // ascending: nothing of this tile behind it
        if (i >= 0) o[i] = LQ ? ((w >> 31) ? -mag : mag) : scale * m.val[k];
    }
}

// A workgroup owns `run` consecutive tiles.  It searches for its part of every message once; from tile to tile it counts
// how many of the pairs it had requested were used, and requests the next ones before it writes the tile.
// G lanes look after one message: 64 for up to four messages, 16 for up to SPARSE_MSGS, so that the searches and the
// loads of all messages are in flight together.
// LQ (Section 4): a kept coordinate decodes to sign * |g|_q, the sign in bit 31 of its index.
// A message whose coordinates do not ascend does not decode (the searches miss some of its pairs): the first `checks`
// workgroups per message compare its neighbours, and latch what they find.  Beside the others, as workgroups of their own: with
// a share of it in every workgroup, 11.17 M outputs took 1.1 us longer.
// AROUND: see AROUND_FROM.
template <bool LQ, bool ACCUMULATE, int G, bool AROUND = false>
__global__ __launch_bounds__(256) void decode_sparse(SparseMsgs msgs, float scale, float* __restrict__ out, long long n, int run,
                                                     int checks, int* flags)
{
    constexpr int EPT = G == 64 ? 2 : 4;                         // pairs per lane requested at once
    __shared__ __attribute__((aligned(16))) float tile[SPARSE_TILE];
    __shared__ long long rest[256 / G];                          // where a message goes on behind those, or -1
    const unsigned int mask = LQ ? 0x7FFFFFFFu : 0xFFFFFFFFu;
    const int tid = threadIdx.x, group = tid / G, glane = tid % G;
    const int shift = (tid & 63) & ~(G - 1);
    const unsigned long long members = G == 64 ? ~0ull : (1ull << (G & 63)) - 1;
    if ((int)blockIdx.x < checks * msgs.n) {
        check_order(msgs.m[blockIdx.x / checks], blockIdx.x % checks, checks, mask, flags);
        return;
    }
    const long long first = (long long)(blockIdx.x - checks * msgs.n) * run * SPARSE_TILE;
    const long long last = min(n, first + (long long)run * SPARSE_TILE);

    const bool mine = group < msgs.n;
    const SparseMsg& m = msgs.m[mine ? group : 0];
    const long long kept = mine ? min(*m.count, m.capacity) : 0;
    const float mag = LQ ? scale * *m.val : 0.0f;
    long long at = lower_bound_group<G>(m.idx, kept, mask, (unsigned int)first);     // first pair that is not in an earlier tile
    unsigned int word[EPT];
    float v[EPT];
    auto request = [&]() {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const long long k = at + glane + G * e;
            word[e] = k < kept ? m.idx[k] : 0u;
            v[e] = LQ ? mag : k < kept ? scale * m.val[k] : 0.0f;
        }
    };
    request();
    for (long long i0 = first; i0 < last; i0 += SPARSE_TILE) {
        const int here = (int)min((long long)SPARSE_TILE, n - i0);
        if (ACCUMULATE) {
            for (int k = tid; k < here; k += 256) tile[k] = out[i0 + k];
        } else {
#pragma unroll
            for (int k = 0; k < SPARSE_TILE / 1024; ++k) *(float4*)&tile[4 * (tid + 256 * k)] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        // which of the requested pairs lie in this tile (a prefix of them: the coordinates ascend)
        bool in[EPT];
        int used = 0;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const long long i = (long long)(word[e] & mask) - i0;
            in[e] = at + glane + G * e < kept && i >= 0 && i < here;
            used += __popcll((__ballot(in[e]) >> shift) & members);
        }
        if (glane == 0) rest[group] = used == G * EPT && at + used < kept ? at + used : -1;
        for (int q = 0; q < msgs.n; ++q) {
            __syncthreads();
            auto put = [&](long long i, float x) { tile[i] = (q == 0 && !ACCUMULATE) ? x : tile[i] + x; };
            if (group == q) {
#pragma unroll
                for (int e = 0; e < EPT; ++e)
                    if (in[e]) put((long long)(word[e] & mask) - i0, LQ && (word[e] >> 31) ? -v[e] : v[e]);
            }
            const long long from = rest[q];
            if (from < 0) continue;
            const SparseMsg& mq = msgs.m[q];
            const long long kept_q = min(*mq.count, mq.capacity);
            const float mag_q = LQ ? scale * *mq.val : 0.0f;
            for (long long k = from + tid; k < kept_q; k += 256) {
                const unsigned int w = mq.idx[k];
                const long long i = (long long)(w & mask) - i0;
                if (i >= here) break;                            // ascending: nothing of this tile behind it
                if (i >= 0) put(i, LQ ? ((w >> 31) ? -mag_q : mag_q) : scale * mq.val[k]);
            }
        }
        if (i0 + SPARSE_TILE < last) {
            // (a message that filled its request is searched for again; the search is entered by whole waves)
            const bool lost = used == G * EPT;
            at += used;
            if (__any(lost)) {
                const long long found = lower_bound_group<G>(m.idx, kept, mask, (unsigned int)(i0 + SPARSE_TILE));
                if (lost) at = found;
            }
            request();
        }
        __syncthreads();
        float* const o = out + i0;
        if (here == SPARSE_TILE && (((size_t)o) & 15) == 0) {
#pragma unroll
            for (int k = 0; k < SPARSE_TILE / 1024; ++k) {
                const floatx4 x = *(const floatx4*)&tile[4 * (tid + 256 * k)];
                if (AROUND) __builtin_nontemporal_store(x, (floatx4*)(o + 4 * (tid + 256 * k)));
                else *(floatx4*)(o + 4 * (tid + 256 * k)) = x;
            }
        } else {
            for (int k = tid; k < here; k += 256) o[k] = tile[k];
        }
        // (the next tile's zeros are written by the thread that has just read the place, as float4 or one by one)
        if (here < SPARSE_TILE || (((size_t)o) & 15) != 0 || ACCUMULATE) __syncthreads();
    }
}

}  // namespace

int decode_svd_batch(atomo_ctx* ctx, const atomo_svd_msg* msgs, const int32_t* first, int n_out, float scale,
                     float* const* outs, const int64_t* lds, bool accumulate, hipStream_t stream)
{
    const int n_msgs = first[n_out];
    std::vector<DecMsg> hm(n_msgs);
    std::vector<DecOut> ho(n_out);
    std::vector<DecWork> hw, hw_tall;
    for (int k = 0; k < n_msgs; ++k)
        hm[k] = DecMsg{msgs[k].count, msgs[k].w, msgs[k].U, msgs[k].V, msgs[k].capacity, 0};
    for (int o = 0; o < n_out; ++o) {
        const atomo_svd_msg& m0 = msgs[first[o]];
        ho[o] = DecOut{outs[o], (long long)lds[o], m0.rows, m0.cols, first[o], first[o + 1]};
        if (m0.cols <= 32 && m0.rows > TR) {
            for (int a = 0; a < (m0.rows + TALL_ROWS - 1) / TALL_ROWS; ++a) hw_tall.push_back(DecWork{o, a, 0, 0});
            continue;
        }
        const int tr = (m0.rows + TR - 1) / TR, tc = (m0.cols + TC - 1) / TC;
        for (int a = 0; a < tr; ++a)
            for (int b = 0; b < tc; ++b) hw.push_back(DecWork{o, a, b, 0});
    }
    // every die gets a contiguous run of the tiles, i.e. the tiles of a few outputs: the singular vectors of an
    // output are then fetched into one L2 instead of all eight
    deal_to_dies(hw);
    deal_to_dies(hw_tall);
    const size_t n_wide = hw.size();
    hw.insert(hw.end(), hw_tall.begin(), hw_tall.end());
    // the three tables in one block; a loop that decodes the same messages into the same outputs finds it on the device
    const size_t at_outs = align_up(hm.size() * sizeof(DecMsg), 256);
    const size_t at_work = align_up(at_outs + ho.size() * sizeof(DecOut), 256);
    std::vector<char>& tables = ctx->table_scratch;
    tables.assign(at_work + hw.size() * sizeof(DecWork), 0);
    memcpy(tables.data(), hm.data(), hm.size() * sizeof(DecMsg));
    memcpy(tables.data() + at_outs, ho.data(), ho.size() * sizeof(DecOut));
    memcpy(tables.data() + at_work, hw.data(), hw.size() * sizeof(DecWork));
    void* d_tables = nullptr;
    const int rc = resident_tables(ctx, ctx->dec_tables, tables, stream, &d_tables);
    if (rc != ATOMO_OK) return rc;
    const DecMsg* d_msgs = (const DecMsg*)d_tables;
    const DecOut* d_outs = (const DecOut*)((char*)d_tables + at_outs);
    const DecWork* d_work = (const DecWork*)((char*)d_tables + at_work);
    {
        ProfScope ps(ctx, ATOMO_K_DECODE_SVD, stream);
        int max_cap = 1;
        for (int k = 0; k < n_msgs; ++k) max_cap = std::max(max_cap, (int)msgs[k].capacity);
        const int batch = std::max(1, ATOMS_MAX / max_cap);      // messages whose atoms fit the LDS list together
        const unsigned grid = (unsigned)hw.size();
        auto launch = [&](auto tall) {
            if (accumulate) decode_svd_tiles<tall, true><<<grid, 256, 0, stream>>>(d_outs, d_msgs, d_work, (int)n_wide, scale, batch);
            else decode_svd_tiles<tall, false><<<grid, 256, 0, stream>>>(d_outs, d_msgs, d_work, (int)n_wide, scale, batch);
        };
        if (hw_tall.empty()) launch(std::false_type());
        else launch(std::true_type());
    }
    ATOMO_HIP(ctx, hipGetLastError());
    return ATOMO_OK;
}

namespace {

// Messages SPARSE_MSGS at a time, in call order; the first launch overwrites the output, the others add to it.
template <bool LQ, typename MSG>
int decode_sparse_all(atomo_ctx* ctx, const MSG* msgs, int n_msgs, float scale, float* out, hipStream_t stream)
{
    const int64_t n = msgs[0].n;
    // one tile per workgroup up to four times what is resident at once (16.8 M outputs: every workgroup starts with a
    // search, but the chip is full); from there on runs of tiles, so that a search serves several
    const int64_t tiles = (n + SPARSE_TILE - 1) / SPARSE_TILE;
    const int run = (int)std::max<int64_t>(1, tiles / SPARSE_RESIDENT / 4);
    // One message's values go behind the zeros (decode_sparse_one) while the zeros are still in a cache: outputs that the L2s hold
    // (16 MB: 1 M outputs 1.03 - 1.28 times faster from 0.1 to 50 % kept, 4 M 1.00 - 1.15), or the last level and few values
    // (11.17 M with 0.1 % 12.2 -> 9.6 us, 1 % 12.9 -> 11.2, but 3 % 13.4 -> 14.3; 33.5 M with 1 % 28.8 -> 24.2, 6 % 33 -> 43).
    // From there on a value costs a read and a write of its line: 67 M with 1 % 52 -> 72 us.
    const bool alone = n_msgs == 1 && (n <= ONE_ANY || (tiles <= ONE_TILES && (int64_t)msgs[0].capacity <= n / 64));
    const unsigned wgs = (unsigned)((tiles + run - 1) / run);
    ProfScope ps(ctx, ATOMO_K_EW_DECODE, stream);
    for (int first = 0; first < n_msgs; first += SPARSE_MSGS) {
        SparseMsgs part = {};
        part.n = std::min(SPARSE_MSGS, n_msgs - first);
        int64_t longest = 0;
        for (int k = 0; k < part.n; ++k) {
            const MSG& m = msgs[first + k];
            longest = std::max(longest, (int64_t)m.capacity);
            if constexpr (LQ) part.m[k] = SparseMsg{(const long long*)m.count, m.idx, m.norm, (long long)m.capacity};
            else part.m[k] = SparseMsg{(const long long*)m.count, m.idx, m.val, (long long)m.capacity};
        }
        // (16 rounds of loads for a workgroup, more from 2 M pairs on, where the tiles take longer than that)
        const int checks = (int)std::min<int64_t>(64, longest / 32768 + 1);
        const unsigned grid = wgs + (unsigned)(checks * part.n);
        if (alone) decode_sparse_one<LQ><<<grid, 256, 0, stream>>>(part.m[0], scale, out, n, checks, ctx->d_flags);
        else if (first > 0) decode_sparse<LQ, true, 16><<<grid, 256, 0, stream>>>(part, scale, out, n, run, checks, ctx->d_flags);
        else if (part.n > 4) decode_sparse<LQ, false, 16><<<grid, 256, 0, stream>>>(part, scale, out, n, run, checks, ctx->d_flags);
        else if (n >= AROUND_FROM) decode_sparse<LQ, false, 64, true><<<grid, 256, 0, stream>>>(part, scale, out, n, run, checks, ctx->d_flags);
        else decode_sparse<LQ, false, 64><<<grid, 256, 0, stream>>>(part, scale, out, n, run, checks, ctx->d_flags);
    }
    ATOMO_HIP(ctx, hipGetLastError());
    return ATOMO_OK;
}

}  // namespace

int decode_entrywise(atomo_ctx* ctx, const atomo_ew_msg* msgs, int n_msgs, float scale, float* out,
                     hipStream_t stream)
{
    return decode_sparse_all<false>(ctx, msgs, n_msgs, scale, out, stream);
}

int decode_lq(atomo_ctx* ctx, const atomo_lq_msg* msgs, int n_msgs, float scale, float* out, hipStream_t stream)
{
    return decode_sparse_all<true>(ctx, msgs, n_msgs, scale, out, stream);
}

}  // namespace atomo
