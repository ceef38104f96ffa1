// Arguments of the matrix-core filter of the grouped scan and of the exact sums of what it lets through.
#pragma once

#include <hip/hip_runtime.h>

#include "ivfpq_lut.hpp"

namespace ivfpq {

constexpr int kFilterPairs = 64;       // pairs of a cluster that one work item takes: two blocks of 32 rows
constexpr int kFilterVectors = 512;    // vectors of the cluster that it takes at most (a multiple of 64 where it takes fewer)

struct FilterArgs {
    const float* queries;         // [nq][d] (tile base), 8-byte aligned
    const float* centroids;
    const float* codebooks;       // [pq_dim][2^bits][m]
    const uint8_t* codes;
    const uint4* pairs;           // [nq][n_probes] {cluster, length, first group, R offset}
    const uint32_t* bounds;       // [nq] per-query upper bound of the k-th smallest R
    const uint32_t* starts;       // [nq] length of a query's list before the filter runs
    uint32_t* counts;             // [nq] length of a query's list
    uint32_t* row_key;            // [nq][stride]: keys (R), behind the nearest probe's segment; the filter leaves the probe's slot here
    uint32_t* row_pos;            // [nq][stride]: positions
    size_t stride;
    const uint4* records;         // the pairs grouped by cluster: {query, slot of the probe, squared distance to the centroid, bound}
    const uint4* items;           // two each: {cluster, first pair, number of pairs, number of vectors}, {first vector, first group, -, -}
    const uint32_t* n_items;
    int nq, n_probes;
    int d, pq_dim, m, bits, code_bytes, chunk_width;
    // R <= bound needs |r - y|^2 <= bound * scale + add + (what saturation may hide); see filter_bound
    float scale, add, top, word_norm_max, eta;
    Fp8Params fp8;                // decode and encode constants of the 8-bit tables
    int truncate;
};

// whether the filter is built for codes of pq_dim fields of `bits` bits over d components, in chunks of `chunk_width` bytes
bool filter_supported(int bits, int pq_dim, int d, int chunk_width);
size_t filter_lds_bytes(int bits, int d);
size_t candidate_lds_bytes(int bits, int d);
int launch_filter(const FilterArgs& a, hipStream_t st);
template <int LUT> int launch_candidates_lut(const FilterArgs& a, hipStream_t st);

}  // namespace ivfpq
