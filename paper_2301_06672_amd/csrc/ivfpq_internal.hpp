// Internal definitions shared by the host-side and device-side halves of libivfpq.
#pragma once

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <new>
#include <string>
#include <thread>
#include <utility>
#include <vector>

#include <sys/mman.h>

#include "../../include/ivfpq.h"

namespace ivfpq {

// Encoding options of one 8-bit table dtype (ivfpq_set_fp8_encoding).
struct Fp8Options {
    int32_t bias;        // exponent bias of the format
    int32_t truncate;    // 0: round to nearest, ties up; 1: truncate
    int32_t per_table;   // 1: the bias is chosen per (query, cluster) table from its largest entry
};

// Launch heuristics a caller may override per index (ivfpq_set_tuning); 0 = the library's own choice.
struct Tuning {
    int32_t scan_threads = 0;   // workgroup size of the scan kernels (64 ... 1024)
    int32_t order_block = 0;    // consecutive pairs of the cluster-grouped order that stay on one XCD
    int32_t scan_share = 0;     // 0: heuristic; 1: one (query, probe) pair per workgroup; 2 or 4: up to that many pairs of a cluster
    int32_t early_exit = 0;     // 0: on (default); 1: on; -1: off (every lookup of Eq. (1) is made)
    int32_t lds_pad = 0;        // extra bytes of LDS requested per scan workgroup (occupancy experiments)
    int32_t scan_route = 0;     // 0: by the amount of work; 1: whole rows; 2: filtered, query by query; 3: filtered, grouped by cluster
};

// Storage of the large host arrays (codes, ids): elements are not cleared when the array is made, since every one of
// them is written right after, and large arrays ask for huge pages (their first touch is what an import costs).
template <class T>
struct HostAllocator {
    using value_type = T;
    static constexpr size_t kHugePage = (size_t)2 << 20;
    HostAllocator() = default;
    template <class U> HostAllocator(const HostAllocator<U>&) {}
    T* allocate(size_t n) {
        if (n > SIZE_MAX / sizeof(T) - kHugePage) throw std::bad_alloc();
        size_t bytes = n * sizeof(T);
        if (bytes < 2 * kHugePage) {
            if (void* p = std::malloc(bytes ? bytes : 1)) return static_cast<T*>(p);
            throw std::bad_alloc();
        }
        bytes = (bytes + kHugePage - 1) / kHugePage * kHugePage;
        void* p = std::aligned_alloc(kHugePage, bytes);
        if (!p) throw std::bad_alloc();
        (void)madvise(p, bytes, MADV_HUGEPAGE);              // advice only: ordinary pages serve as well
        return static_cast<T*>(p);
    }
    void deallocate(T* p, size_t) { std::free(p); }
    template <class U> void construct(U* p) { ::new (static_cast<void*>(p)) U; }
    template <class U, class... Args> void construct(U* p, Args&&... args) { ::new (static_cast<void*>(p)) U(std::forward<Args>(args)...); }
    template <class U> bool operator==(const HostAllocator<U>&) const { return true; }
    template <class U> bool operator!=(const HostAllocator<U>&) const { return false; }
};
template <class T> using HostArray = std::vector<T, HostAllocator<T>>;

// memcpy by a few threads: one thread is bound by the page faults of a destination that is touched for the first time
// (48 MB into new memory: 3.6 ms by one thread)
inline void copy_bytes(void* dst, const void* src, size_t bytes) {
    constexpr size_t kPerThread = (size_t)2 << 20;
    const size_t hw = std::thread::hardware_concurrency();
    size_t parts = bytes / kPerThread;
    parts = parts > 8 ? 8 : parts;
    parts = parts > hw ? hw : parts;
    if (parts < 2) {
        if (bytes) std::memcpy(dst, src, bytes);
        return;
    }
    const size_t step = (bytes / parts + kPerThread - 1) / kPerThread * kPerThread;   // no huge page is touched by two
    std::thread pool[8];
    size_t at = step;                                        // the first part is this thread's own
    try {
        for (size_t t = 1; t < parts && at < bytes; ++t) {
            const size_t len = t + 1 == parts || bytes - at < step ? bytes - at : step;
            pool[t] = std::thread([=] { std::memcpy((char*)dst + at, (const char*)src + at, len); });
            at += len;
        }
    } catch (...) {                                          // no more threads to be had: the rest is copied below
    }
    std::memcpy(dst, src, step);
    if (at < bytes) std::memcpy((char*)dst + at, (const char*)src + at, bytes - at);
    for (auto& t : pool)
        if (t.joinable()) t.join();
}

// Of a search for 1, 2, 4 ... 64 probes: how many clusters' ranking values are within their error bound of what a selection by waves takes as
// its limit, the mean of a sample.  Few where distances differ by more than the bound, which goes with the squared norms; many where
// the vectors share an offset.
struct RankCrowd {
    static constexpr int kRanks = 7;
    float within[kRanks] = {};
    float of(int n_probes) const {
        int rank = 0;
        while (rank + 1 < kRanks && (1 << rank) < n_probes) ++rank;
        return within[rank];
    }
};

// The share of a farther cluster's vectors that pass the matrix-core filter, a property of the indexed vectors that their number does
// not tell: lists that overlap pass many times what lists apart from each other do.  Sampled from the saved index: for clusters at
// ranks 1, 2, 4, ... from a query, bounds of k / length = share, and limits wider than the bound by looseness.
struct PassShares {
    static constexpr int kRanks = 9, kShares = 7, kLoose = 4;
    static constexpr float share(int s) {
        constexpr float v[kShares] = {0.01f, 0.02f, 0.05f, 0.1f, 0.2f, 0.5f, 1.f};
        return v[s];
    }
    static constexpr float looseness(int i) {
        constexpr float v[kLoose] = {0.01f, 0.04f, 0.07f, 0.13f};
        return v[i];
    }
    int ranks = 0;                                 // how many ranks there are figures for; 0: none
    float pass[kRanks][kShares][kLoose] = {};
};

// Device image of an index.  All pointers point into the single buffer the caller handed to
// ivfpq_upload; the library owns none of them.
struct DeviceImage {
    bool valid = false;
    int device = -1;
    const float* centroids = nullptr;      // [n_lists][d]
    const float* centroid_norms = nullptr; // [n_lists] squared L2 norms
    const float* codebooks = nullptr;      // [pq_dim][ksub][m]
    const int64_t* list_offsets = nullptr; // [n_lists+1], unpadded vector offsets (into ids)
    const uint32_t* list_sizes = nullptr;  // [n_lists]
    const float* list_radii = nullptr;     // [n_lists] largest squared norm of a cluster's decoded residuals
    const int64_t* group_offsets = nullptr;// [n_lists+1], offsets in 64-vector groups (into codes)
    const uint8_t* codes = nullptr;        // interleaved, see ivfpq_upload
    const int64_t* ids = nullptr;          // [n] list order
};

}  // namespace ivfpq

struct ivfpq_index {
    int64_t n = 0;
    int32_t d = 0, n_lists = 0, pq_dim = 0, pq_bits = 0;
    std::vector<float> centroids;       // [n_lists][d]
    std::vector<float> codebooks;       // [pq_dim][2^pq_bits][d/pq_dim]
    std::vector<int64_t> list_offsets;  // [n_lists+1]
    ivfpq::HostArray<uint8_t> codes;    // [n][code_bytes], list order
    ivfpq::HostArray<int64_t> ids;      // [n], list order

    // derived at import
    int64_t total_groups = 0;           // sum over lists of ceil(len/64)
    std::vector<uint32_t> sorted_padded_sizes;  // padded list lengths, descending
    double list_mean = 0.0, list_typical = 0.0; // length of a list that is not empty; of the list that a vector lies in (sum of len^2 / n)

    ivfpq::DeviceImage dev;
    ivfpq::Fp8Options fp8_opt[2] = {{15, 0, 0}, {7, 0, 0}};   // e5m3, e4m4 (ivfpq_set_fp8_encoding)
    float centroid_norm_max = 0.f;      // largest squared centroid norm (set by ivfpq_upload)
    float word_norm_max = -1.f;         // largest codeword norm (set by ivfpq_upload); negative: some codeword is not a moderate number
    ivfpq::PassShares pass_shares;      // set by ivfpq_upload
    ivfpq::RankCrowd rank_crowd;        // set by ivfpq_upload
    size_t workspace_limit = (size_t)32 << 30;   // search scratch (R, positions, ranking values) per query tile

    ivfpq::Tuning tuning;               // ivfpq_set_tuning

    // stage timing (hipEvent_t kept as void* so this header stays free of HIP types).  Search calls take the
    // handle as const and record into these: with timing enabled, calls on one index must not overlap.
    bool timing = false;
    mutable bool stage_valid = false;
    struct Span { void* a; void* b; int stage; float share; };    // share: the part of the time between the events that is the stage's
    mutable std::vector<void*> event_pool;
    mutable std::vector<Span> spans;
    mutable size_t events_used = 0;
    mutable char scan_kernel[256] = {};      // what the last timed search launched for the probes other than the nearest (ivfpq_scan_kernel_info)
    mutable int scan_kernel_lut = -1;        // its table dtype; -1: no such launch

    int32_t ksub() const { return 1 << pq_bits; }
    int32_t m() const { return d / pq_dim; }
    int32_t code_bytes() const { return pq_dim * pq_bits / 8; }
    // upper bound of (padded) candidates one query can see with n_probes probes
    int64_t max_padded_candidates(int32_t n_probes) const {
        int64_t s = 0;
        for (int32_t i = 0; i < n_probes && i < (int32_t)sorted_padded_sizes.size(); ++i)
            s += sorted_padded_sizes[i];
        return s;
    }
};

namespace ivfpq {

RankCrowd sample_rank_crowd(const ivfpq_index& idx, float centroid_norm_max) noexcept;
// of an index of at most 128 components; none otherwise
PassShares sample_pass_shares(const ivfpq_index& idx) noexcept;
// The share for a search: averaged over ranks 1 .. n_probes - 1, linear between the sampled ranks, in log(share) and in the looseness.
double pass_share(const PassShares& p, int n_probes, double share, double loose);

// Work on a thread of its own, or on this one where there is none to be had.  It must not throw; the destructor waits for it.
class SideTask {
public:
    template <class F>
    explicit SideTask(F work) {
        try {
            thread_ = std::thread(work);
        } catch (...) {
            work();
        }
    }
    ~SideTask() { wait(); }
    SideTask(const SideTask&) = delete;
    SideTask& operator=(const SideTask&) = delete;
    void wait() { if (thread_.joinable()) thread_.join(); }

private:
    std::thread thread_;
};

void set_error(const char* fmt, ...);
int fail(int status, const char* fmt, ...);

// Runs `body` (-> int status) and turns a C++ exception into a status: nothing throws across the C ABI.
template <class Body>
int guarded(const char* what, Body&& body) {
    try {
        return body();
    } catch (const std::bad_alloc&) {
        return fail(IVFPQ_ENOSPACE, "%s: out of host memory", what);
    } catch (const std::exception& e) {
        return fail(IVFPQ_EINVAL, "%s: %s", what, e.what());
    } catch (...) {
        return fail(IVFPQ_EINVAL, "%s: unknown exception", what);
    }
}

// validates shape parameters common to build and import; returns IVFPQ_OK or sets the error
int check_shape(int64_t n, int32_t d, int32_t n_lists, int32_t pq_dim, int32_t pq_bits);

// fills the derived fields after the logical arrays are in place
void finish_import(ivfpq_index* idx);

// SplitMix64: the generator behind every seeded draw of the builders
struct SplitMix64 {
    uint64_t s;
    explicit SplitMix64(uint64_t seed) : s(seed) {}
    uint64_t next() {
        uint64_t z = (s += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    }
    uint64_t below(uint64_t bound) { return next() % bound; }
};

// `k` start rows out of `n` (ascending): distinct when n >= k, cycling otherwise
std::vector<int64_t> draw_rows(SplitMix64& rng, int64_t n, int k);
// at most `limit` rows of [0, n) at a fixed stride (all rows when n <= limit)
std::vector<int64_t> stride_rows(int64_t n, int64_t limit);

// called by ivfpq_free before the handle goes away (destroys HIP events); defined in the device half
void release_device_state(ivfpq_index* idx);

}  // namespace ivfpq
