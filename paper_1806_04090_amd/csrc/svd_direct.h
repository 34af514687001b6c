// Direct Spectral-ATOMO encode (svd_direct.hip, svd_direct_values.hip): descriptors and launches shared with the host side in svd.hip.
#pragma once

#include "svd_common.h"

namespace atomo {
namespace direct {

constexpr int MAX_R = 640;           // vectors on the shorter side that the reduction holds in registers
constexpr int TILE = 64;
constexpr int RB = 16;               // reflectors per block of the way back through H
// a wave takes a tile of the Gram product of its own (direct_gram_wide) in calls with so many such work items, of chunks of so many
// columns
constexpr size_t WIDE_MIN = 8192;
constexpr int WIDE_COLUMNS = 256;
constexpr double MAX_BUDGET = 32.0;  // above this many expected atoms the vectors cost more than the Jacobi iteration
constexpr long long START_TICKS = 2000000;   // 20 ms of the 100 MHz clock: how long a workgroup waits for its group to start

// State words of a matrix (device, int32).
enum {
    DS_ACCEPT = 0,       // 1: the message is in place and the Jacobi iteration leaves the matrix alone
    DS_EXP = 1,          // the Gram matrix was multiplied by 2^-DS_EXP (even) before the reduction
    DS_FAIL = 2,         // 1: a wait of the reduction hit its bound (the matrix is not accepted)
    DS_ZERO_ROWS = 3,    // rows of A that are exactly zero
    DS_BROKEN = 4,       // 1: the message is no decomposition of the matrix: a kept vector was not accepted, or DS_FAIL
                         //    (DS_ACCEPT is 0 then)
    DS_WORDS = 8
};

struct DirectMat {
    const float* G;
    long long ldg;
    int rows, cols, transposed, r, M;
    int nt, pad;                     // N = 64 nt >= r: the Gram matrix with `pad` zero rows and columns in front
    int cls;                         // CLS_*: how the reduction splits the matrix (its last rows are one workgroup's)
    int nchunks, kchunk;             // the columns of A in the Gram product: nchunks partial sums of kchunk each
    int capacity;
    double* part;                    // [nchunks][nt (nt + 1) / 2][64 * 64] partial Gram tiles
    double* C;                       // [N][N] Gram matrix, both triangles
    double* diag;                    // [N] its diagonal: the squared norms of the rows of A
    double* refl;                    // [N][N] row k: the Householder vector of step k (entries from 64 (k / 64) on)
    double* tau;                     // [N]
    double2* td;                     // [N] tridiagonal matrix, scaled: squared coupling to the entry before (kept above
                                     //   OD2_MIN), diagonal; (0, 2) in the padding
    double* od;                      // [N] couplings: od[k] between k and k + 1
    double* fact;                    // [N / 16][16][16] triangular factors of the blocks of 16 reflectors
    double* lam;                     // [r] eigenvalues, descending, scaled
    double* fine;                    // [r] where in its cell of the search each of them is
    double* u;                       // [capacity][r] kept vectors of the shorter side
    unsigned long long* xch;         // exchange slots of the reduction, see Tri
    double* half;                    // [3][384] where one group leaves the reduction to another: the column, and the last step's vectors
    unsigned long long* gate;        // [2] the workgroups that have started, of the matrix's group and of one of eight, see Gate
    unsigned* tickets;               // [nt (nt + 1) / 2] chunks of a tile that are done, see direct_gram_wide
    int* st;                         // [DS_WORDS]
    int* count;
    int* idx;
    float* w;
    float* U;
    float* V;
    float* sigma_out;                // may be null
    float* p_out;                    // may be null
    float* weight;                   // [capacity] weight sigma / p of the kept atom (folded messages: it goes into U)
    unsigned long long stream_id;
    int* report;                     // [2] sweeps (1: solved directly) and passes over the data
    int index;                       // which matrix of the call this is
    int alone;                       // 1: no iteration behind it, so it is reported if it is not accepted
};

struct DirectPlan {
    std::vector<DirectMat> mats;
    std::vector<svd::Work> gram, tiles, gram_wide, tri, tri_half, eig, vec, lng;
    bool spread = false;             // deal the workgroups of a group over all dies (for tests)
    long long start_ticks = START_TICKS;
    int eig_lanes = 32;              // lanes per eigenvalue in the search, at most 32
    bool few = false, half = false;  // reduction: direct_tridiagonal_few takes `tri`; behind direct_tridiagonal_half with `tri_half`
    size_t n_eig = 0;                // how many items of `eig` are searches; the others are blocks of reflectors
    int max_nt = 1;
    size_t n_work() const { return gram.size() + tiles.size() + gram_wide.size() + tri.size() + tri_half.size() + eig.size() + vec.size() + lng.size(); }
};

// Lets the kernels have more LDS than a launch gets by default; once per device.
hipError_t allow_lds();
// true if a matrix of r vectors on the shorter side is of a size for this path
bool eligible(int r);
// Lays out one matrix (base of `carve` null: sizes only).
void plan_matrix(Carver& carve, DirectMat& m);
void plan_work(DirectPlan& plan);

struct DirectTables {
    const DirectMat* mats;
    int n_mats;
    const svd::Work *gram, *tiles, *gram_wide, *tri, *tri_half, *eig, *vec, *lng;
};
// hint_out (may be null, has to be if anything iterates): where the words for the next calls go.  gram_done (may be null) is recorded
// behind the Gram products; if that fails nothing else is enqueued.  done (may be null) is recorded behind the last kernel.
hipError_t launch(const DirectPlan& plan, const DirectTables& t, double s, uint64_t seed, int* hint_out, int* d_flags, hipStream_t stream,
                  hipEvent_t gram_done, hipEvent_t done);
// its part in svd_direct_values.hip
void launch_eigenvalues(const DirectPlan& plan, const DirectTables& t, hipStream_t stream);

}  // namespace direct
}  // namespace atomo
