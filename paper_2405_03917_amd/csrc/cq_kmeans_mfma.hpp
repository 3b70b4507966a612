// Lloyd iterations for groups of 256 centroids (cq_kmeans_mfma.hip).
#pragma once

#include "cq_internal.hpp"

namespace cq {

struct KMeansLloyd {
    const uint16_t* xg;       // fp16 [G][n][c]
    const uint32_t* wq;       // [G][n] integer weights, or null: all tokens weigh the same
    float* cent;              // fp32 [G][256][c], updated in place
    uint16_t* assign;         // [G][n] assignment of the last iteration, or null
    void* scratch;            // for the sums of token splits; may be small (fewer splits then)
    size_t scratch_bytes;
    int groups, n, n_iter;
};
cq_status launch_kmeans_lloyd(const KMeansLloyd& a, int c, hipStream_t stream);

}  // namespace cq
