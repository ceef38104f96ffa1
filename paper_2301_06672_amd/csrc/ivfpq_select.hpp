// Exact selection by one workgroup (k-th smallest key, k smallest records), and the small wave-level sums and scans
// it uses.  Included by .hip translation units only; everything has internal linkage.
#pragma once

#include <hip/hip_runtime.h>

#include "ivfpq_lds_util.hpp"
#include "ivfpq_rank.hpp"

namespace {

constexpr uint32_t kPadKey = 0xFFFFFFFFu;      // R of a padding lane: sorts after every real distance

// ================================================================================================
// Exact selection of the k smallest of n keyed elements by one workgroup.
// Keys are the bit patterns of non-negative floats (order-preserving as unsigned integers); equal
// keys are ordered by a signed 64-bit tie key, then by position.  MSB-first radix select with 8-bit
// digits finds the k-th smallest key; everything below it and the needed share of the ties is
// collected into LDS records and sorted there (bitonic).
// ================================================================================================
// (the helpers below are force-inlined: left to the inliner, a few lines more in one of them turned it into a
// real call with its arguments on the stack, and the probe-selection kernel took twice as long)
constexpr int SEL_THREADS = 256;
constexpr int SEL_CAP = 1024;      // record capacity = IVFPQ_MAX_K: the selected elements always fit

// what block_kth_key alone needs
struct KthShared {
    uint32_t hist[256];
    uint32_t digit, need, count;
    uint32_t n_rec;
};

// CAP: how many records the selection can return (>= k); kernels whose k is small take a small CAP, so that more of
// their workgroups share a compute unit (they wait on barriers and memory most of the time: the top-k kernel with
// k = 100 took 0.25 ms at six workgroups per compute unit and 0.21 ms at eight)
template <int CAP>
struct SelectSharedT {
    static constexpr int kCap = CAP;
    uint32_t hist[256];
    uint32_t rec_key[CAP];
    uint32_t rec_pos[CAP];
    long long rec_tie[CAP];
    uint32_t digit, need, count;   // broadcast slots of the digit search
    uint32_t n_rec, n_eq;
};
using SelectShared = SelectSharedT<SEL_CAP>;
constexpr int SEL_CAP_SMALL = 256;  // >= 2 * kFewMax: block_select_few parks tie keys in the upper half of the records

// The sum of a value over every aligned group of 8 lanes, left in all 8: neighbours, then pairs inside a quad, then
// the other quad of the group (whose four lanes hold the same value by then, so the mirrored order does not matter).
// Each step adds the same two numbers in both partners: all 8 lanes end with the same bits.
__device__ inline float sum_over_8_lanes(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));     // quad_perm [1,0,3,2]
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));     // quad_perm [2,3,0,1]
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true));    // row_half_mirror
    return v;
}

// Sum over this lane and the lanes below it, by data-parallel permutes (no trip through the LDS): a scan inside
// every row of 16 lanes, then the last lane of a row added to the rows above.  (A lane a permute has no source
// for, or whose row is masked out, receives 0.)
template <int CTRL, int ROWS>
__device__ inline uint32_t dpp_or_zero(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, true); }
__device__ inline uint32_t wave_inclusive_scan(uint32_t v) {
    v += dpp_or_zero<0x111, 0xF>(v);       // row_shr:1
    v += dpp_or_zero<0x112, 0xF>(v);       // row_shr:2
    v += dpp_or_zero<0x114, 0xF>(v);       // row_shr:4
    v += dpp_or_zero<0x118, 0xF>(v);       // row_shr:8
    v += dpp_or_zero<0x142, 0xA>(v);       // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xC>(v);       // row_bcast:31 into rows 2 and 3
    return v;
}

// hist holds digit counts; finds the digit that contains the `need`-th smallest element
// (1-based).  Result in s.digit (the digit), s.need (rank inside that digit), s.count (its count).
// Called by all threads; contains barriers.
template <class Shared>
__device__ __forceinline__ void find_digit(Shared& s, uint32_t need) {
    __syncthreads();
    if (threadIdx.x < kWave) {
        const int t = threadIdx.x;
        uint32_t c0 = s.hist[4 * t], c1 = s.hist[4 * t + 1], c2 = s.hist[4 * t + 2], c3 = s.hist[4 * t + 3];
        uint32_t sum = c0 + c1 + c2 + c3;
        uint32_t incl = wave_inclusive_scan(sum);
        uint32_t excl = incl - sum;
        if (excl < need && need <= incl) {
            uint32_t r = need - excl, dsel = 0, cnt = c0;
            if (r > c0) { r -= c0; dsel = 1; cnt = c1;
                if (r > c1) { r -= c1; dsel = 2; cnt = c2;
                    if (r > c2) { r -= c2; dsel = 3; cnt = c3; } } }
            s.digit = 4 * t + dsel;
            s.need = r;
            s.count = cnt;
        }
    }
    __syncthreads();
}

__device__ inline bool rec_less(uint32_t ka, long long ta, uint32_t pa, uint32_t kb, long long tb, uint32_t pb) {
    if (ka != kb) return ka < kb;
    if (ta != tb) return ta < tb;
    return pa < pb;
}

// sorts records [0, np2) ascending by (key, tie, pos); np2 is a power of two <= the record capacity
template <class S>
__device__ __forceinline__ void sort_records(S& s, int np2) {
    for (int size = 2; size <= np2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            __syncthreads();
            for (int t = threadIdx.x; t < (np2 >> 1); t += blockDim.x) {
                int lo = ((t / stride) * stride * 2) + (t % stride);
                int hi = lo + stride;
                bool up = ((lo & size) == 0);
                uint32_t ka = s.rec_key[lo], kb = s.rec_key[hi];
                long long ta = s.rec_tie[lo], tb = s.rec_tie[hi];
                uint32_t pa = s.rec_pos[lo], pb = s.rec_pos[hi];
                bool b_lt_a = rec_less(kb, tb, pb, ka, ta, pa);
                if (b_lt_a == up) {
                    s.rec_key[lo] = kb; s.rec_key[hi] = ka;
                    s.rec_tie[lo] = tb; s.rec_tie[hi] = ta;
                    s.rec_pos[lo] = pb; s.rec_pos[hi] = pa;
                }
            }
        }
    }
    __syncthreads();
}

// One histogram increment per active lane, with the increments of a wave folded into a single
// LDS atomic when all its active lanes hit the same bin (the usual case for the leading digit of
// distances of similar magnitude, where per-lane atomics on one address would serialise).
__device__ __forceinline__ void hist_add(uint32_t* hist, uint32_t digit, bool active) {
    const unsigned long long act = ballot64(active);
    if (act == 0) return;
    const int first = __ffsll((long long)act) - 1;
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)digit, first);      // `first` is the same for the whole wave
    const unsigned long long same = ballot64(active && digit == d0);
    if (same == act) {
        if ((int)(threadIdx.x & (kWave - 1)) == first) atomicAdd(&hist[d0], (uint32_t)__popcll(act));
    } else if (active) {
        atomicAdd(&hist[digit], 1u);
    }
}

// The kk-th smallest (1-based, 1 <= kk <= n) of n keys, by four 8-bit digits from the top.
// *rank_in_ties = how many elements equal to the result rank at or below kk (1..*n_ties),
// *n_ties = number of elements equal to the result.  Called by every thread of the workgroup.
template <class Shared, class KeyFn>
__device__ __forceinline__ uint32_t block_kth_key(Shared& s, uint32_t n, uint32_t kk, KeyFn key_of,
                                  uint32_t* rank_in_ties, uint32_t* n_ties) {
    const int tid = threadIdx.x, nth = blockDim.x;
    uint32_t prefix = 0, need = kk, n_eq = 0;
    for (int pass = 3; pass >= 0; --pass) {
        const int shift = pass * 8;
        __syncthreads();
        for (int b = tid; b < 256; b += nth) s.hist[b] = 0;
        __syncthreads();
        for (uint32_t base = 0; base < n; base += nth) {
            const uint32_t i = base + tid;
            const bool valid = i < n;
            const uint32_t key = valid ? key_of(i) : 0u;
            const bool in = valid && ((pass == 3) || ((key >> (shift + 8)) == (prefix >> (shift + 8))));
            hist_add(s.hist, (key >> shift) & 255u, in);
        }
        find_digit(s, need);
        prefix |= s.digit << shift;
        need = s.need;
        n_eq = s.count;
    }
    *rank_in_ties = need;
    *n_ties = n_eq;
    return prefix;
}

// How keys stand for floats: the bit pattern itself (distances, never negative) or the monotone map of ordered_key.  Keys from
// kNotFinite on are infinities, not-a-numbers and padding; below zero, the ordered map's negative ones.
struct PlainKey {
    static constexpr uint32_t kNotFinite = 0x7F800000u;
    static __device__ float value(uint32_t key) { return __uint_as_float(key); }
    static __device__ uint32_t key(float v) { return __float_as_uint(v); }
    static __device__ bool finite(uint32_t key) { return key < kNotFinite; }
};
struct OrderedKey {
    static __device__ float value(uint32_t key) { return ordered_key_value(key); }
    static __device__ uint32_t key(float v) { return ordered_key(v); }
    static __device__ bool finite(uint32_t key) { return key < 0xFF800000u && key > 0x007FFFFFu; }
};

// Equal bins over the values of a set of keys.
constexpr int kBins = 256;
struct Bins {
    float from, inv, width, to;
    bool usable;                 // some keys are finite and their range has a width
    template <class K>
    __device__ int of(uint32_t key) const {
        if (!K::finite(key)) return kBins - 1;
        const int b = (int)((K::value(key) - from) * inv);
        return b < kBins - 1 ? b : kBins - 1;
    }
};

// Histogram of n keys (s.hist) over equal bins between the least and the largest finite one; not-finite keys fall into the last bin.
// The numbering is monotone in the key.  Called by every thread; ends with a barrier.
template <class K, class Shared, class KeyFn>
__device__ __forceinline__ Bins bin_histogram(Shared& s, uint32_t n, KeyFn key_of) {
    const int tid = threadIdx.x, nth = blockDim.x;
    uint32_t lo = 0xFFFFFFFFu, hi = 0;
    for (uint32_t i = tid; i < n; i += nth) {
        const uint32_t key = key_of(i);
        if (K::finite(key)) { lo = lo < key ? lo : key; hi = hi > key ? hi : key; }
    }
    __syncthreads();
    if (tid == 0) { s.digit = 0xFFFFFFFFu; s.need = 0u; }
    for (int b = tid; b < kBins; b += nth) s.hist[b] = 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t l2 = (uint32_t)__shfl_xor((int)lo, off, kWave), h2 = (uint32_t)__shfl_xor((int)hi, off, kWave);
        lo = lo < l2 ? lo : l2;
        hi = hi > h2 ? hi : h2;
    }
    __syncthreads();
    if ((tid & (kWave - 1)) == 0) { atomicMin(&s.digit, lo); atomicMax(&s.need, hi); }
    __syncthreads();
    Bins bins;
    bins.from = K::value(s.digit);
    bins.to = K::value(s.need);
    bins.usable = s.digit < s.need;
    bins.width = (bins.to - bins.from) * (1.f / (kBins - 1));
    bins.usable = bins.usable && bins.width > 0.f && bins.width < 3.0e38f;
    bins.inv = bins.usable ? 1.f / bins.width : 0.f;
    if (bins.usable)
        for (uint32_t i = tid; i < n; i += nth) atomicAdd(&s.hist[bins.of<K>(key_of(i))], 1u);
    __syncthreads();
    return bins;
}

// A key not below the kk-th smallest (1 <= kk <= n), close to it: the upper edge of the bin that holds it, or the exact key where the bin
// holds many others.  Three barriers for a histogram instead of the four rounds of block_kth_key; for callers that need a bound only.
template <class K, class Shared, class KeyFn>
__device__ __forceinline__ uint32_t block_kth_bound(Shared& s, uint32_t n, uint32_t kk, KeyFn key_of) {
    const Bins bins = bin_histogram<K>(s, n, key_of);
    uint32_t r0, r1;
    if (bins.usable) {
        find_digit(s, kk);
        const uint32_t bin = s.digit, in_bin = s.count;
        if (bin < kBins - 1 && in_bin <= 32u + kk / 4u) {
            // the roundings of a bin's number and of its edge stay within a few 2^-22 of the range or of the value
            const float edge = bins.from + (float)(bin + 1) * bins.width * 1.000002f;
            const float up = edge + __builtin_fabsf(edge) * 5.0e-7f;
            __syncthreads();
            return K::key(up < bins.to ? up : bins.to);
        }
        __syncthreads();
    }
    return block_kth_key(s, n, kk, key_of, &r0, &r1);
}

// The selection of block_select_smallest by bins: elements of the bins up to the one that holds the kk-th are collected bin by bin,
// each then counts the elements of its own bin that precede it.  Seven barriers instead of some forty (four rounds of digits, a bitonic
// sort).  Returns 0, with nothing selected, where bins do not spread the keys: ties, values that cluster, a few far outliers.
template <class S, class KeyFn, class TieFn>
__device__ __forceinline__ int block_select_bins(S& s, uint32_t n, uint32_t kk, KeyFn key_of, TieFn tie_of) {
    const int tid = threadIdx.x, nth = blockDim.x;
    constexpr uint32_t kMost = 64;                       // elements of a bin: the count inside it is quadratic
    const Bins bins = bin_histogram<PlainKey>(s, n, key_of);
    if (!bins.usable) return 0;
    if (tid < kWave) {
        uint32_t c[kBins / kWave], sum = 0, most = 0;
#pragma unroll
        for (int u = 0; u < kBins / kWave; ++u) { c[u] = s.hist[tid * (kBins / kWave) + u]; sum += c[u]; }
        uint32_t at = wave_inclusive_scan(sum) - sum;
        if (tid == 0) s.count = 0;
#pragma unroll
        for (int u = 0; u < kBins / kWave; ++u) {
            s.hist[tid * (kBins / kWave) + u] = at;      // the bin's first record
            if (at < kk) {
                most = most > c[u] ? most : c[u];
                if (kk <= at + c[u]) { s.digit = (uint32_t)(tid * (kBins / kWave) + u); s.need = at + c[u]; }
            }
            at += c[u];
        }
        if (ballot64(most > kMost) != 0 && tid == 0) s.count = 1;
    }
    __syncthreads();
    const uint32_t last = s.digit, total = s.need;
    if (s.count != 0 || total > (uint32_t)S::kCap || last == (uint32_t)kBins - 1u) { __syncthreads(); return 0; }
    for (uint32_t i = tid; i < n; i += nth) {
        const uint32_t key = key_of(i);
        const uint32_t b = (uint32_t)bins.of<PlainKey>(key);
        if (b <= last) {
            const uint32_t slot = atomicAdd(&s.hist[b], 1u);       // in the end the next bin's first record
            s.rec_key[slot] = key; s.rec_pos[slot] = i; s.rec_tie[slot] = tie_of(i);
        }
    }
    __syncthreads();
    constexpr int kEach = (S::kCap + SEL_THREADS - 1) / SEL_THREADS;      // records a thread ranks (workgroups of SEL_THREADS or more)
    uint32_t key[kEach], pos[kEach], rank[kEach];
    long long tie[kEach];
#pragma unroll
    for (int e = 0; e < kEach; ++e) {
        const uint32_t r = (uint32_t)tid + (uint32_t)(e * nth);
        rank[e] = 0xFFFFFFFFu;
        if (r >= total) continue;
        key[e] = s.rec_key[r]; pos[e] = s.rec_pos[r]; tie[e] = s.rec_tie[r];
        const int b = bins.of<PlainKey>(key[e]);
        const uint32_t first = b ? s.hist[b - 1] : 0u, end = s.hist[b];
        uint32_t before = first;
        for (uint32_t j = first; j < end; ++j) before += rec_less(s.rec_key[j], s.rec_tie[j], s.rec_pos[j], key[e], tie[e], pos[e]) ? 1u : 0u;
        rank[e] = before;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kEach; ++e)
        if (rank[e] < kk) { s.rec_key[rank[e]] = key[e]; s.rec_pos[rank[e]] = pos[e]; s.rec_tie[rank[e]] = tie[e]; }
    __syncthreads();
    return (int)kk;
}

// KeyFn(i) -> uint32 key of element i; TieFn(i) -> long long tie key of element i.
// On return records [0, min(k, n)) hold the selected elements in ascending (key, tie, pos) order.
// Returns min(k, n).  Must be called by every thread of the workgroup.
template <class S, class KeyFn, class TieFn>
__device__ __forceinline__ int block_select_smallest(S& s, uint32_t n, uint32_t k, KeyFn key_of, TieFn tie_of) {
    const uint32_t kk = k < n ? k : n;
    if (kk == 0) return 0;
    const int tid = threadIdx.x, nth = blockDim.x;
    if (const int got = block_select_bins(s, n, kk, key_of, tie_of)) return got;

    uint32_t need = 0, n_eq = 0;
    const uint32_t T = block_kth_key(s, n, kk, key_of, &need, &n_eq);
    const uint32_t n_less = kk - need;     // elements strictly below T: all selected

    // ---- collect
    __syncthreads();
    if (tid == 0) { s.n_rec = 0; s.n_eq = 0; }
    __syncthreads();
    const bool all_fit = (n_less + n_eq) <= (uint32_t)S::kCap;
    if (all_fit) {
        // everything <= T goes into the records; the sort decides which ties stay
        for (uint32_t i = tid; i < n; i += nth) {
            uint32_t key = key_of(i);
            if (key <= T) {
                uint32_t slot = atomicAdd(&s.n_rec, 1u);
                s.rec_key[slot] = key; s.rec_pos[slot] = i; s.rec_tie[slot] = tie_of(i);
            }
        }
    } else {
        // too many elements equal to T: pick the `need` smallest tie keys among them with a second,
        // 64-bit radix select (tie keys mapped to unsigned order by flipping the sign bit)
        unsigned long long uprefix = 0;
        uint32_t uneed = need;
        for (int pass = 7; pass >= 0; --pass) {
            const int shift = pass * 8;
            __syncthreads();
            for (int b = tid; b < 256; b += nth) s.hist[b] = 0;
            __syncthreads();
            for (uint32_t base = 0; base < n; base += nth) {
                const uint32_t i = base + tid;
                bool in = i < n && key_of(i) == T;
                unsigned long long u = 0;
                if (in) {
                    u = (unsigned long long)tie_of(i) ^ 0x8000000000000000ull;
                    in = (pass == 7) || ((u >> (shift + 8)) == (uprefix >> (shift + 8)));
                }
                hist_add(s.hist, (uint32_t)(u >> shift) & 255u, in);
            }
            find_digit(s, uneed);
            uprefix |= (unsigned long long)s.digit << shift;
            uneed = s.need;
        }
        // uprefix = the need-th smallest tie key; uneed = how many copies of it to take
        __syncthreads();
        for (uint32_t i = tid; i < n; i += nth) {
            uint32_t key = key_of(i);
            if (key > T) continue;
            bool take = key < T;
            long long tie = tie_of(i);
            if (!take) {
                unsigned long long u = (unsigned long long)tie ^ 0x8000000000000000ull;
                if (u < uprefix) take = true;
                else if (u == uprefix) take = atomicAdd(&s.n_eq, 1u) < uneed;
            }
            if (take) {
                uint32_t slot = atomicAdd(&s.n_rec, 1u);
                s.rec_key[slot] = key; s.rec_pos[slot] = i; s.rec_tie[slot] = tie;
            }
        }
    }
    __syncthreads();
    const uint32_t n_rec = s.n_rec;
    int np2 = 1;
    while ((uint32_t)np2 < n_rec) np2 <<= 1;
    for (int i = n_rec + tid; i < np2; i += nth) {
        s.rec_key[i] = 0xFFFFFFFFu; s.rec_pos[i] = 0xFFFFFFFFu; s.rec_tie[i] = 0x7FFFFFFFFFFFFFFFll;
    }
    sort_records(s, np2);
    return (int)kk;
}

// The same selection for few elements (n <= kFewMax <= blockDim.x; key_of must be cheap, every thread
// calls it n times): thread i ranks element i by counting the elements that precede it in (key, tie,
// index) order, three barriers in all.  It costs about n instructions per thread where the radix select
// and the sort cost several hundred whatever n is.  Tie keys are fetched only for elements with fewer than
// k smaller keys, and wait in the upper half of the record array while the ranks are settled.
constexpr uint32_t kFewMax = 128;
template <class S, class KeyFn, class TieFn>
__device__ __forceinline__ int block_select_few(S& s, uint32_t n, uint32_t k, KeyFn key_of, TieFn tie_of) {
    static_assert(S::kCap >= 2 * (int)kFewMax, "tie keys wait in the upper half of the records");
    const uint32_t kk = k < n ? k : n;
    if (kk == 0) return 0;
    const uint32_t e = threadIdx.x;
    constexpr uint32_t SCR = S::kCap / 2;
    __syncthreads();
    const uint32_t key = e < n ? key_of(e) : 0xFFFFFFFFu;
    uint32_t less = 0, same = 0;
    if (e < n)
        for (uint32_t j = 0; j < n; ++j) {
            const uint32_t kj = key_of(j);
            less += kj < key ? 1u : 0u;
            same += kj == key ? 1u : 0u;
        }
    const bool cand = e < n && less < kk;
    long long tie = 0;
    if (cand) { tie = tie_of(e); s.rec_tie[SCR + e] = tie; }
    __syncthreads();
    if (cand) {
        uint32_t r = less;
        if (same > 1)                        // elements with the same key all have their tie key in place
            for (uint32_t j = 0; j < n; ++j) {
                if (j == e || key_of(j) != key) continue;
                const long long tj = s.rec_tie[SCR + j];
                r += (tj < tie || (tj == tie && j < e)) ? 1u : 0u;
            }
        if (r < kk) { s.rec_key[r] = key; s.rec_tie[r] = tie; s.rec_pos[r] = e; }
    }
    __syncthreads();
    return (int)kk;
}

// ------------------------------------------------------------------------------------------------
// The k smallest of a long row of keys in global memory (tens of thousands per query).
// The k-th smallest key among the first CAND_CAP elements is an upper bound of the k-th smallest
// of the whole row, so one streaming pass that keeps only keys not above that bound compacts the
// row into LDS (typically a few times k elements); the exact selection then runs on that small
// set.  If the compacted set overflows LDS the routine falls back to exact selection over the
// whole row in global memory.  tie_of_pos(pos, key) gives the tie key of the element at row
// position pos.  On return records [0, got) hold key, tie and row position in ascending
// (key, tie) order.
// ------------------------------------------------------------------------------------------------
constexpr int CAND_CAP = 1024;   // >= IVFPQ_MAX_K

template <int CAP>
struct RowSelectSharedT {
    SelectSharedT<CAP> sel;
    uint32_t cand_key[CAND_CAP];
    uint32_t cand_pos[CAND_CAP];
    uint32_t n_cand;
};
using RowSelectShared = RowSelectSharedT<SEL_CAP>;

// K: what the keys stand for (PlainKey, OrderedKey).
// pos_of(i): logical position of row element i (what the records report and what tie_of_pos
// takes); have_bound/bound: an upper bound of the k-th smallest key that the caller already knows
// (at least k elements of the row are <= it).
// Hooks for rows whose keys are only approximate (probe selection): widen(bound) is applied to every
// bound before it filters (it must return a key that no element the exact selection could need
// exceeds); refine(n_cand) runs once the candidates sit in LDS, may replace their keys by exact ones and
// drop candidates (it returns how many remain, at the front of the candidate arrays); whole_row() is the
// fallback when compaction fails and must return the selection itself.
struct NoWiden { __device__ uint32_t operator()(uint32_t b) const { return b; } };
struct NoRefine { __device__ uint32_t operator()(uint32_t n) const { return n; } };

template <class K, class T, class PosFn, class TieFn, class WidenFn, class RefineFn, class WholeRowFn>
__device__ __forceinline__ int block_select_row_ex(T& t, const uint32_t* __restrict__ row, uint32_t n, uint32_t k,
                                   bool have_bound, uint32_t bound, PosFn pos_of, TieFn tie_of_pos,
                                   WidenFn widen, RefineFn refine, WholeRowFn whole_row) {
    auto& s = t.sel;
    const int tid = threadIdx.x, nth = blockDim.x;
    const uint32_t kk = k < (uint32_t)CAND_CAP ? k : (uint32_t)CAND_CAP;
    bool compact = true;
    uint32_t n_cand = n;
    __syncthreads();
    if (n > (uint32_t)CAND_CAP) {
        uint32_t r0, r1;
        if (!have_bound) {
            // the k-th smallest of the first S keys bounds the k-th smallest of the row; about k n / S keys
            // pass it, so S grows with k n until half the LDS buffer is the expectation (a second pass
            // over the whole row costs more than a longer sample)
            const unsigned long long want = (unsigned long long)kk * n / (CAND_CAP / 2);
            const uint32_t S = want <= (unsigned long long)CAND_CAP ? (uint32_t)CAND_CAP : (want < n ? (uint32_t)want : n);
            if (S == (uint32_t)CAND_CAP) {
                for (int i = tid; i < CAND_CAP; i += nth) t.cand_key[i] = row[i];
                bound = block_kth_bound<K>(s, (uint32_t)CAND_CAP, kk, [&](uint32_t i) { return t.cand_key[i]; });
            } else {
                bound = block_kth_bound<K>(s, S, kk, [&](uint32_t i) { return row[i]; });
            }
        }
        bound = widen(bound);
        const bool vec = (reinterpret_cast<uintptr_t>(row) & 15u) == 0;      // 16-byte loads, the last n % 4 keys one by one
        compact = false;
        // Each pass keeps the elements not above the bound.  If they overflow the LDS buffer, the
        // k-th smallest of the ones that were kept is a tighter valid bound (they are all members
        // of the row): the survivor count shrinks by about CAND_CAP / k per pass.
        for (int pass = 0; pass < 8; ++pass) {
            __syncthreads();
            if (tid == 0) t.n_cand = 0;
            __syncthreads();
            auto keep = [&](uint32_t key, uint32_t i) {
                if (key <= bound) {
                    uint32_t slot = atomicAdd(&t.n_cand, 1u);
                    if (slot < (uint32_t)CAND_CAP) { t.cand_key[slot] = key; t.cand_pos[slot] = pos_of(i); }
                }
            };
            if (vec) {
                const uint4* row4 = reinterpret_cast<const uint4*>(row);
                for (uint32_t i4 = tid; i4 < n / 4; i4 += nth) {
                    const uint4 v = row4[i4];
                    keep(v.x, i4 * 4); keep(v.y, i4 * 4 + 1); keep(v.z, i4 * 4 + 2); keep(v.w, i4 * 4 + 3);
                }
                for (uint32_t i = (n & ~3u) + tid; i < n; i += nth) keep(row[i], i);
            } else {
                for (uint32_t i = tid; i < n; i += nth) keep(row[i], i);
            }
            __syncthreads();
            n_cand = t.n_cand;
            if (n_cand <= (uint32_t)CAND_CAP) { compact = true; break; }
            const uint32_t tighter = widen(block_kth_key(s, (uint32_t)CAND_CAP, kk, [&](uint32_t i) { return t.cand_key[i]; }, &r0, &r1));
            if (tighter >= bound) break;      // a plateau of equal keys: no progress possible this way
            bound = tighter;
        }
    } else {
        for (uint32_t i = tid; i < n; i += nth) { t.cand_key[i] = row[i]; t.cand_pos[i] = pos_of(i); }
        __syncthreads();
    }
    int got;
    if (compact) {
        n_cand = refine(n_cand);
        auto key_of = [&](uint32_t i) { return t.cand_key[i]; };
        auto tie_of = [&](uint32_t i) -> long long { return tie_of_pos(t.cand_pos[i], t.cand_key[i]); };
        got = n_cand <= kFewMax ? block_select_few(s, n_cand, k, key_of, tie_of)
                                : block_select_smallest(s, n_cand, k, key_of, tie_of);
        for (int j = tid; j < got; j += nth) s.rec_pos[j] = t.cand_pos[s.rec_pos[j]];   // back to logical positions
    } else {
        got = whole_row();
    }
    __syncthreads();
    return got;
}

template <class T, class PosFn, class TieFn>
__device__ __forceinline__ int block_select_row(T& t, const uint32_t* __restrict__ row, uint32_t n, uint32_t k,
                                bool have_bound, uint32_t bound, PosFn pos_of, TieFn tie_of_pos) {
    auto& s = t.sel;
    return block_select_row_ex<PlainKey>(t, row, n, k, have_bound, bound, pos_of, tie_of_pos, NoWiden{}, NoRefine{},
        [&]() -> int {
            const int got = block_select_smallest(s, n, k,
                [&](uint32_t i) { return row[i]; },
                [&](uint32_t i) -> long long { return tie_of_pos(pos_of(i), row[i]); });
            for (int j = threadIdx.x; j < got; j += blockDim.x) s.rec_pos[j] = pos_of(s.rec_pos[j]);
            return got;
        });
}

}  // namespace
