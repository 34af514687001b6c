// Spectral-ATOMO encode of thin matrices (svd_thin.hip): descriptors and launches shared with the host side in svd.hip.
#pragma once

#include "svd_common.h"

namespace atomo {
namespace thin {

using svd::THIN_R;

struct ThinMat {
    const float* G;
    long long ldg;
    int rows, cols, tall, r, M;
    int nchunks, chunk;              // the positions of the long side in partial Gram matrices of `chunk` each
    int capacity;
    double* part;                    // [nchunks][3][16 * 16]: the tiles (0, 0), (1, 0), (1, 1) of the partial sums, of which
                                     //   the entries of the lower triangle are read (up to 16 columns: the first)
    double* u;                       // [r + 8][r] kept vectors of the shorter side, divided by their sigma (folded: times the weight
                                     //   where the longer side is U)
    int* count;
    int* idx;
    float* w;
    float* U;
    float* V;
    float* sigma_out;                // may be null
    float* p_out;                    // may be null
    unsigned long long stream_id;
    int* report;                     // [2] sweeps (1: solved directly) and passes over the data
};

struct ThinPlan {
    std::vector<ThinMat> mats;
    std::vector<svd::Work> gram, lng;
    size_t n_work() const { return gram.size() + lng.size(); }
};

// Lays one matrix out (base of `carve` null: sizes only); plan_work lists the work of all.
void plan_matrix(Carver& carve, ThinMat& m);
void plan_work(ThinPlan& plan);
// done (may be null) is recorded behind the last kernel
hipError_t launch(const ThinPlan& plan, const ThinMat* d_mats, const svd::Work* gram, const svd::Work* lng, double s, uint64_t seed,
                  int* d_flags, hipStream_t stream, hipEvent_t done);

}  // namespace thin
}  // namespace atomo
