// Internal declarations shared by the translation units of libatomo (gfx950 only).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <tuple>
#include <vector>

#include "../../include/atomo.h"
#include "../../include/atomo_bench.h"
#include "../../include/atomo_debug.h"

namespace atomo {

// ---------------------------------------------------------------------------------------------
// Context
// ---------------------------------------------------------------------------------------------

// Device-side latched flags (int32 each).
enum { FLAG_CAPACITY = 0, FLAG_NOCONV = 1, FLAG_MAX_SWEEPS = 2, FLAG_EIG_VISITS = 3, FLAG_EIG_INNER = 4, FLAG_DS_UPDATE_UNITS = 5, FLAG_ORDER = 6, FLAG_COUNT = 8 };

// How an SVD encode goes about a matrix: Jacobi iteration; direct encode with the iteration behind it for what that leaves
// over; direct encode alone.
enum : uint8_t { ROUTE_ITERATE = 0, ROUTE_BOTH = 1, ROUTE_DIRECT = 2 };

// Events between streams of this device, and one that tells the host that a kernel has ended whose words for it are fenced: without
// the flush to the host and to other devices that an event makes otherwise.  Between two kernels of a stream such an event takes
// 1.1 us, with that flush 3.
// HIP describes the flag for events that only take the time, whose inspection by the host need not synchronise with the work in front
// of them.  What is relied on here is less than that and more: the host's words are fenced in the kernel that writes them
// (__threadfence_system), and what a stream finds behind hipStreamWaitEvent rests on the release of device scope that every kernel
// ends with and the acquire that the next one begins with, by which the kernels of one stream see each other's results on other dies too.
// The latter is how the runtime works (ROCm 7, one device) and not a promise of the flag; it does not reach memory of other devices.
constexpr unsigned ON_DEVICE_EVENT = hipEventDisableTiming | hipEventDisableSystemFence;

// What an SVD encode learnt about its matrices, for the calls after it (atomo_svd_options.adaptive).
constexpr int HINT_MATS = 4;     // word of the first matrix
struct SweepHint {
    int32_t* host = nullptr;     // pinned, device-visible: [0] most sweeps of a Gram-space matrix, [1] of a data-space one,
                                 // [2] 1 once written, [3] see ask_from, [HINT_MATS + j] 1 if matrix j was solved directly
    int32_t* dev = nullptr;      // the same memory as the device addresses it
    size_t cap = 0;              // words
    hipEvent_t done = nullptr;   // recorded after the kernel that writes `host`
    bool pending = false;        // the event has not been seen complete yet
    uint64_t sig = 0;            // shapes of the call
    uint64_t seq = 0;            // order of the calls (0 = unused)
    int limit_gs = 0, limit_ds = 0;   // the sweep limits that call ran with
    std::vector<uint8_t> route;  // ROUTE_* of every matrix
    std::vector<uint8_t> passed; // calls in a row that have not tried to solve the matrix, which an earlier one could not
    bool iterated = false;       // the iteration was enqueued: `host` holds sweep counts of the matrices that it had
};

// Descriptor tables that the device holds, with what they were made from.  They hold addresses, sizes and stream ids, never
// data, so a call whose tables come out byte for byte like one of these uploads nothing.  Four of them: a program that
// goes through a few sets of buffers in turn (one per worker, double buffering) finds each where it left it.
struct TableSlot {
    void* dev = nullptr;
    size_t cap = 0;
    std::vector<char> host;
    hipStream_t stream = nullptr;
    uint64_t used = 0;
};
struct TableCache {
    TableSlot slot[4];
    uint64_t clock = 0;
};

struct StageSlot {
    void* host = nullptr;        // pinned
    size_t bytes = 0;
    hipEvent_t ev = nullptr;     // recorded after the last copy out of `host`
    bool pending = false;
};

}  // namespace atomo

struct atomo_ctx {
    int device = 0;
    void* ws = nullptr;          // device workspace
    size_t ws_bytes = 0;
    size_t ws_refused = SIZE_MAX;    // smallest workspace with the direct encode's part that could not be had (atomo_reserve forgets it)
    int32_t* d_flags = nullptr;  // [FLAG_COUNT] device
    int32_t* h_flags = nullptr;  // pinned readback buffer
    int last_hip = 0;
    atomo::StageSlot ring[8];
    int ring_next = 0;
    // sweep and refresh counts of the last SVD encode, [2 * report_n] on the device, outside the workspace (which the
    // next call of any kind overwrites)
    int32_t* d_report = nullptr;
    size_t report_cap = 0;               // pairs allocated
    size_t report_n = 0;                 // matrices of the last SVD encode
    // streams and events of the SVD encoder's internal fork/join (created on first use, default priority)
    void* ew_state = nullptr;            // entry-wise encoder: search state kept from call to call (histograms zero between calls)
    atomo::SweepHint hints[4];
    int hint_next = 0;
    uint64_t hint_seq = 0;
    bool direct_lds = false;       // direct::allow_lds has been called for this context's device
    bool direct_spread = false;            // atomo_debug_direct_groups
    long long direct_start_ticks = -1;     // (negative: the library's own bound)
    int ew_spins = -1;                     // atomo_debug_entrywise_counts (negative: the library's own bound)
    size_t rowgram_lds = 0;        // dynamic LDS that svd_rowgram has been allowed on this context's device
    atomo::TableCache svd_tables, dec_tables, prob_tables;   // of the SVD encoder, the SVD decoder and atomo_probabilities
    std::vector<char> table_scratch;     // where a call puts its tables together
    hipStream_t side = nullptr, side2 = nullptr, side_thin = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr, ev_join2 = nullptr, ev_join_thin = nullptr;
    // optional event bracketing of kernel launches (atomo_profile_*)
    bool profiling = false;
    std::vector<hipEvent_t> ev_pool;     // pairs: [2k] start, [2k+1] stop
    std::vector<int> ev_kind;            // kernel class of pair k
    size_t ev_used = 0;                  // pairs in use
};

namespace atomo {

#define ATOMO_HIP(ctx, call)                                   \
    do {                                                       \
        hipError_t e__ = (call);                               \
        if (e__ != hipSuccess) {                               \
            (ctx)->last_hip = (int)e__;                        \
            return ATOMO_EHIP;                                 \
        }                                                      \
    } while (0)

// Grows the workspace to at least `bytes` (contents are not preserved).
int ensure_workspace(atomo_ctx* ctx, size_t bytes);

// Creates the context's side streams and the fork/join events if they do not exist yet.
int ensure_side_streams(atomo_ctx* ctx);

// Copies `bytes` of host data to device address `dst` on `stream` through a pinned staging slot,
// so the caller's host buffer may be reused as soon as this returns.
int upload(atomo_ctx* ctx, void* dst, const void* src, size_t bytes, hipStream_t stream);

// Where on the device `tables` are (uploaded on `stream`, in place of the set that has not been used for longest, if no
// set of the cache is the same).
int resident_tables(atomo_ctx* ctx, TableCache& cache, const std::vector<char>& tables, hipStream_t stream, void** dev);

// Brackets the launches issued during its lifetime with two events when profiling is on.
struct ProfScope {
    atomo_ctx* ctx;
    hipStream_t stream;
    hipEvent_t stop = nullptr;
    ProfScope(atomo_ctx* c, int kind, hipStream_t s) : ctx(c), stream(s)
    {
        if (!ctx->profiling) return;
        if (ctx->ev_used * 2 >= ctx->ev_pool.size()) {
            hipEvent_t a = nullptr, b = nullptr;
            if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) return;
            ctx->ev_pool.push_back(a);
            ctx->ev_pool.push_back(b);
            ctx->ev_kind.push_back(kind);
        }
        ctx->ev_kind[ctx->ev_used] = kind;
        (void)hipEventRecord(ctx->ev_pool[ctx->ev_used * 2], stream);
        stop = ctx->ev_pool[ctx->ev_used * 2 + 1];
        ++ctx->ev_used;
    }
    ~ProfScope()
    {
        if (stop) (void)hipEventRecord(stop, stream);
    }
};

// Launches a kernel and records `done` (may be null) behind it, as the completion of the kernel itself where the stream is not being
// captured: a record of its own is one more packet between this kernel and the next, 1.1 us.
template <typename... P, typename... A>
hipError_t launch_recorded(hipEvent_t done, void (*kernel)(P...), unsigned grid, unsigned block, size_t lds, hipStream_t stream, A... args)
{
    if (done) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusActive;
        if (hipStreamIsCapturing(stream, &capture) != hipSuccess) (void)hipGetLastError();
        if (capture == hipStreamCaptureStatusNone) {
            std::tuple<P...> values(args...);
            return std::apply([&](auto&... x) {
                void* at[] = {(void*)&x...};
                return hipExtLaunchKernel((const void*)kernel, dim3(grid), dim3(block), at, lds, stream, nullptr, done, 0);
            }, values);
        }
    }
    kernel<<<grid, block, lds, stream>>>(args...);
    return done ? hipEventRecord(done, stream) : hipSuccess;
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// A bump allocator over the workspace; first pass with base == nullptr only measures.
struct Carver {
    char* base;
    size_t off = 0;
    size_t last = 0;                     // offset of what the last take returned
    explicit Carver(void* b) : base((char*)b) {}
    template <typename T>
    T* take(size_t count) {
        off = align_up(off, 256);
        last = off;
        T* p = base ? (T*)(base + off) : nullptr;
        off += count * sizeof(T);
        return p;
    }
};

// Workgroups go to the chip's eight dies in turn (workgroup b to die b mod 8), and each die has its own L2.  Reorders a
// work list so that every die gets one contiguous run of it: neighbours in the list, which read the same operands,
// then find them in the same L2 instead of fetching them into all eight.
template <typename T>
inline void deal_to_dies(std::vector<T>& list)
{
    constexpr size_t DIES = 8;
    const size_t n = list.size();
    std::vector<T> dealt(n);
    size_t start[DIES + 1] = {0};
    for (size_t x = 0; x < DIES; ++x) start[x + 1] = start[x] + (n + DIES - 1 - x) / DIES;
    for (size_t b = 0; b < n; ++b) dealt[b] = list[start[b % DIES] + b / DIES];
    list.swap(dealt);
}

// What a lane loads from LDS behind this is what other lanes of its wave stored in front of it.  The wave's LDS operations are performed in
// program order, so there is nothing to wait for, but without the fences the compiler may keep a lane's own value or move the load: the
// barrier alone says nothing of memory.
__device__ inline void lanes_in_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): device + host inline so every kernel draws the same stream
// ---------------------------------------------------------------------------------------------

struct u32x4 { uint32_t x, y, z, w; };

// One instruction (the compiler makes two of a ^ b ^ c): 18 of the 34 exclusive-ors of a block's rounds go.
__host__ __device__ inline uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
    return a ^ b ^ c;
#endif
}

__host__ __device__ inline u32x4 philox4x32_10(uint64_t block, uint64_t stream_id, uint64_t seed)
{
    uint32_t c0 = (uint32_t)block, c1 = (uint32_t)(block >> 32);
    uint32_t c2 = (uint32_t)stream_id, c3 = (uint32_t)(stream_id >> 32);
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return u32x4{c0, c1, c2, c3};
}

// 24 random bits -> [0,1), exact in float32.
__host__ __device__ inline float u01(uint32_t word) { return (float)(word >> 8) * 5.9604644775390625e-08f; }

// ---------------------------------------------------------------------------------------------
// Entry points implemented per translation unit
// ---------------------------------------------------------------------------------------------

int svd_workspace_bytes(const atomo_mat* mats, int n_mats, size_t* bytes);
int encode_svd(atomo_ctx* ctx, const atomo_mat* mats, int n_mats, double s, uint64_t seed, uint64_t stream_base,
               const atomo_svd_options* opt, const atomo_svd_msg* msgs, float* sigma_out, float* p_out,
               hipStream_t stream);

int svd_sweeps(atomo_ctx* ctx, hipStream_t stream, int32_t* sweeps, int32_t* refreshes, int n_mats);

size_t entrywise_workspace_bytes(int64_t n);
int encode_entrywise(atomo_ctx* ctx, const float* g, double s, uint64_t seed, uint64_t stream_id,
                     const atomo_ew_msg* msg, float* p_out, hipStream_t stream);
int entrywise_noalloc_setup(atomo_ctx* ctx);   // device address of the static scratch array, once per device
int encode_lq(atomo_ctx* ctx, const float* g, double q, uint64_t seed, uint64_t stream_id, const atomo_lq_msg* msg,
              float* p_out, hipStream_t stream);
int probabilities(atomo_ctx* ctx, const float* lambda, const int64_t* offsets, int n_seg, double s, float* p,
                  hipStream_t stream);

// accumulate: outs[o] += ... instead of outs[o] = ...
int decode_svd_batch(atomo_ctx* ctx, const atomo_svd_msg* msgs, const int32_t* first, int n_out, float scale,
                     float* const* outs, const int64_t* lds, bool accumulate, hipStream_t stream);
int decode_entrywise(atomo_ctx* ctx, const atomo_ew_msg* msgs, int n_msgs, float scale, float* out,
                     hipStream_t stream);
int decode_lq(atomo_ctx* ctx, const atomo_lq_msg* msgs, int n_msgs, float scale, float* out, hipStream_t stream);

}  // namespace atomo
