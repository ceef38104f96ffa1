// Arguments of the scan kernels, and the launch of those that take several pairs of a cluster per workgroup.
#pragma once

#include <hip/hip_runtime.h>

#include "ivfpq_lut.hpp"

namespace ivfpq {

struct ScanArgs {
    const float* queries;         // [nq][d] (tile base)
    const float* centroids;
    const float* codebooks;
    const uint32_t* list_sizes;
    const int64_t* group_offsets;
    const uint8_t* codes;
    const uint4* pairs;           // [nq][n_probes] {cluster, length, first group, R offset}; unused in single-list mode
    uint32_t* bounds;             // [nq] per-query upper bound of the k-th smallest R: written by mode 1, read in filtered mode
    uint32_t* counts;             // [nq] survivors appended so far (begun by mode 1, extended in filtered mode)
    uint32_t* starts;             // [nq] mode 1: their number when it ends, or null
    uint32_t* Rpos;               // [nq][stride] row position of each appended survivor (filtered mode)
    Fp8Mode fp8;                  // encoding of the 8-bit table dtypes (unused by the other two)
    int mode;                     // 1: nearest probe of every query, every R written in place; 3: the same for all probes;
                                  // 2: the other probes, only R <= bound appended behind the nearest probe's segment
    float* R;                     // [nq][stride]
    size_t stride;
    int n_probes;
    int n_lists;
    int d, pq_dim, m, bits;
    int n_chunks;                 // chunks per vector (code_bytes / CW)
    int single_list;              // >= 0: scan this cluster for query 0, R written from offset 0
    const uint32_t* order;        // mode 2: pairs (as q * (n_probes - 1) + probe - 1) grouped by cluster, or null; mode 1 of the group kernel: queries
                                  // in the order of their nearest clusters
    uint32_t n_pairs;             // number of entries of the order
    uint32_t order_block;         // consecutive ones that stay on one XCD
    int k_bound;                  // mode 1: the k of the bound to take from the nearest probe's values; 0: none is wanted
    uint32_t* clear[2];           // mode 1: counters of the grouping that follows, n_clear[] words each, to be set to zero
    uint32_t n_clear[2];
    int early_exit;               // mode 2: stop adding for a 64-vector group once every partial sum is over the bound
};

constexpr uint32_t kAdmitAll = 0xFFFFFFFEu;   // a bound: every real R is below this, the padding key is above
constexpr int kAliveCap = 64;        // groups of a wave that the first pass of the split scan can note for the second
constexpr int kGroupStageAll = 128;  // survivors a wave stages before it appends them, over all queries of a run: 128 / R per query
                                     // (a 64-vector group with more survivors than that goes straight to the list)
constexpr int kGroupHead = 128;      // bytes at the start of the kernel's LDS that hold the slot's pair descriptors

// scan_group_kernel over a.n_pairs pairs, up to G of a cluster per workgroup (ivfpq_scan_group.hip, one object per LUT).  Mode 1: the nearest
// probes of the queries a.order[0 .. n_pairs), all values written in place.
template <int LUT>
int launch_scan_group_kernel(const ScanArgs& a, int G, int threads, size_t lds, hipStream_t st);

}  // namespace ivfpq
