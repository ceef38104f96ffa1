// Device half of libivfpq: upload of the index image and the HIP kernels of the IVFPQ search phase
// (arXiv 2301.06672, Sec. I-C second enumeration, Sec. I-D, Sec. II) for gfx950 (MI355X, wave64).
//
// Kernels, in the order one search call runs them (per tile of queries):
//   coarse_rank_*_kernel step 1a: ranking values |c|^2 - 2 q.c of every (query, cluster) pair on the
//                        matrix cores: bf16 instructions on operands split in two for large problems,
//                        fp32 otherwise; stored as all keys (few clusters) or as the three smallest
//                        tagged keys of every strip of 32 / 64 clusters
//   cluster_distance_kernel  few queries instead: the exact distances, which step 1b then selects from as they are
//   select_probes_kernel step 1b: candidates by ranking value with a rigorous error bound, exact
//                        direct-form distances for them, exact selection of the n_probes nearest
//                        clusters; per-pair descriptors and R offsets (select_probes_wave_kernel: a wave per query, ivfpq_probe_wave.hpp)
//   (large batches: nearest_order_kernel, scan_group_kernel of up to four queries and bound_wave_kernel take the next one's place)
//   scan_kernel (mode 1) steps 2-4 for the nearest probe of every query: query residual, lookup table F
//                        built in LDS as fp32 / half / e5m3 / e4m4, then every wave streams 64-vector
//                        groups of PQ codes from HBM and accumulates R = sum_j F(y_j) (Eq. 1)
//                        and, at its end, a bound a little above the k-th smallest R of that cluster, hence above the final
//                        k-th distance of the query; the cluster's values under it start the survivor list
//   pair_count / pair_offsets / pair_scatter   the other (query, probe) pairs grouped by cluster
//                        (counts per workgroup in LDS first when there are few clusters)
//   scan_kernel (mode 2) steps 2-4 for the other probes, in cluster-grouped, XCD-aware order (a
//                        cluster's codes then come from one XCD's L2); only R values under the bound
//                        are kept
//   scan_group_kernel    the same for up to four neighbouring pairs of one cluster per workgroup (8- and 4-bit codes, 32
//                        to 96 sub-spaces of the others):
//                        their tables are interleaved entry by entry, so one LDS read serves one lookup of
//                        every query of the group; codebooks and codes are read once for all of them
//   scan_filter_kernel / candidate_kernel   large batches instead: a matrix product lists the vectors that can have R <= bound, and
//                        only those are added up (ivfpq_scan_filter.hip, ivfpq_candidates.hip); filter_items_kernel lays out its work
//   topk_kernel          step 5: the k smallest R among the survivors of a query, ordered by
//                        (R, id), and the map from (cluster, position) to the caller's ids
// Where little is scanned in all (scan_route), launches count more than the work they save: the filtered scan takes its
// pairs in query order, and below that scan_kernel (mode 3) writes the values of all probes for the top-k step to read.
// Beside the path: dump_lut_kernel (steps 2-3 of one pair, for inspection) and refine_kernel (exact
// re-ranking of candidates with the stored vectors).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <utility>

#include "ivfpq_filter_bound.hpp"
#include "ivfpq_internal.hpp"
#include "ivfpq_bound_wave.hpp"
#include "ivfpq_rank.hpp"
#include "ivfpq_lds_util.hpp"
#include "ivfpq_lut.hpp"
#include "ivfpq_probe_wave.hpp"
#include "ivfpq_scan_args.hpp"
#include "ivfpq_scan_filter.hpp"
#include "ivfpq_select.hpp"

using namespace ivfpq;

// The workspace of ivfpq_search_static: a fixed device array, so that callers who cannot allocate (HIP graph
// capture, serving loops, harnesses that forbid hipMalloc) need bring none.  Each GPU the library runs on holds
// its own copy at its own address until the process ends.  In host code this name is only a stand-in for the
// symbol: the array's device address comes from hipGetSymbolAddress (static_scratch_ptr), and only that pointer
// is ever handed to kernels.
static __device__ __align__(256) unsigned char scratch[IVFPQ_STATIC_SCRATCH_BYTES];

namespace {

constexpr size_t kStaticScratchBytes = IVFPQ_STATIC_SCRATCH_BYTES;

// Device address of `scratch` on the current device, looked up once per device.
int static_scratch_ptr(void** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* ptr[kMaxDevices] = {};
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(IVFPQ_EUNSUPPORTED, "device ordinal %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(IVFPQ_EHIP, "hipGetSymbolAddress gave a null address for the static scratch");
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return IVFPQ_OK;
}

// ================================================================================================
// Step 1b: probe selection for one query per workgroup: short-list by the ranking values of step
// 1a (with their error bound), exact distances for the short list, exact selection among those.
// Also lays out the query's slice of the R scratch: roff[p] = first slot of probe p, roff[n_probes]
// = padded candidate count (every cluster padded to a multiple of 64 vectors), and writes one
// descriptor per (query, probe) pair -- {cluster, length, first 64-vector group, R offset} -- so
// that a scan workgroup starts from a single 16-byte load.
// S (may be null): instead of the keys, the ranking kernel's summary of every strip of strip_w clusters
// (its three smallest keys, tagged with the cluster's position in the strip), strip-major
// [n_strips][gridDim.x]; the host passes it when there are at least 2 n_probes strips.  The n_probes-th
// smallest strip minimum then bounds the n_probes-th smallest key; a strip whose minimum passes the
// (widened) bound yields its best cluster, its best two if the second key passes too, or all its clusters if
// the third does as well, and all of
// these get their exact distance.  A is then only scratch for the whole-row fallback.
// ================================================================================================
// CAP: record capacity, >= n_probes.  The small one serves selections from strip summaries only (S given): the path
// that streams all keys short-lists up to CAND_CAP indices in the record arrays.
template <int CAP, int THREADS, bool EXACT = false>
__global__ void __launch_bounds__(THREADS)
select_probes_kernel(uint32_t* __restrict__ A, const StripSummary* __restrict__ S, int strip_w,
                     const float* __restrict__ queries,
                     const float* __restrict__ centroids, float centroid_norm_max, int d,
                     int n_lists, int n_probes,
                     const uint32_t* __restrict__ list_sizes, const int64_t* __restrict__ group_offsets,
                     uint32_t* __restrict__ probes, float* __restrict__ probe_dists,
                     uint32_t* __restrict__ roff, uint4* __restrict__ pairs, int k_hint, uint32_t* __restrict__ nearest) {
    __shared__ RowSelectSharedT<CAP> t;
    __shared__ float s_part[THREADS / kWave];
    auto& s = t.sel;
    // Workgroup b runs on XCD b % 8.  Inside every block of 64 queries the eight workgroups of one XCD take eight
    // consecutive queries: their strip summaries (16 bytes per query and strip, strip-major) share 128-byte lines,
    // so a line is fetched into one XCD's L2 instead of all eight.
    const int b = blockIdx.x;
    const int q = b < (int)(gridDim.x & ~63u) ? (b & ~63) + ((b & 7) << 3) + ((b >> 3) & 7) : b;
    const int tid = threadIdx.x, nth = blockDim.x;
    const int lane = tid & (kWave - 1), wave = tid >> 6, n_waves = nth >> 6;
    const float* qv = queries + (size_t)q * d;
    uint32_t* row = A + (size_t)q * n_lists;       // ranking keys of a(q, c) = |c|^2 - 2 q.c

    auto wave_sum = [&](float v) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
        return v;
    };
    // |q|^2, for the error bound of a()
    float part = 0.f, qn = 0.f;
    if (S) {             // (the strip minima go the same way, see below: their loads travel with the query's)
        const uint32_t n_strips = ((uint32_t)n_lists + strip_w - 1) / strip_w;
        if (n_strips <= (uint32_t)CAND_CAP)
            for (uint32_t i = tid; i < n_strips; i += nth) t.cand_key[i] = S[q + i * (size_t)gridDim.x].x;
    }
    if constexpr (!EXACT) {
        for (int c = tid; c < d; c += nth) part = __builtin_fmaf(qv[c], qv[c], part);
        part = wave_sum(part);
        if (lane == 0) s_part[wave] = part;
        __syncthreads();
        for (int w = 0; w < n_waves; ++w) qn += s_part[w];
    }
    // |a_computed - a_exact| <= delta
    const float delta = rank_error_bound(d, qn, centroid_norm_max);
    // keys up to this one can belong to a cluster whose exact rank is within the bound's rank
    auto widen = [&](uint32_t key) {
        const float f = ordered_key_value(key);
        float g = f + 2.f * delta;
        g += __builtin_fabsf(g) * 2.3841858e-07f;          // the addition above rounds: stay on the safe side
        return (g == g) ? ordered_key(g) : 0xFFFFFFFFu;     // NaN (from infinite inputs): admit everything
    };
    // exact squared distance to cluster l (direct form) by a group of 8 adjacent lanes: each lane sums
    // every 8th component, then three exchange steps; the order is fixed, so the value of a cluster
    // does not depend on which path computes it.  Every lane of the group gets the result.
    auto exact8 = [&](uint32_t l, bool valid) {
        float acc = 0.f;
        if (valid) {
            const float* c = centroids + (size_t)l * d;
            for (int u = tid & 7; u < d; u += 8) { const float diff = qv[u] - c[u]; acc = __builtin_fmaf(diff, diff, acc); }
        }
        acc = sum_over_8_lanes(acc);
        return acc;
    };
    // n of them, cluster_of(j), each to sink(j, distance) in the first lane of its group; two per group at a time, so that the loads of
    // both are under way together
    auto exact_all = [&](uint32_t n, auto cluster_of, auto sink) {
        const uint32_t per = nth / 8;
        for (uint32_t base = 0; base < n; base += 2 * per) {
            const uint32_t j0 = base + (tid >> 3), j1 = j0 + per;
            const bool v0 = j0 < n, v1 = j1 < n;
            const float *c0 = centroids + (size_t)(v0 ? cluster_of(j0) : 0u) * d, *c1 = centroids + (size_t)(v1 ? cluster_of(j1) : 0u) * d;
            float a0 = 0.f, a1 = 0.f;
            if (v0) {
#pragma unroll 4
                for (int u = tid & 7; u < d; u += 8) {
                    const float x = qv[u], d0 = x - c0[u], d1 = x - c1[u];
                    a0 = __builtin_fmaf(d0, d0, a0);
                    a1 = __builtin_fmaf(d1, d1, a1);
                }
            }
            a0 = sum_over_8_lanes(a0);
            a1 = sum_over_8_lanes(a1);
            if ((tid & 7) == 0) {
                if (v0) sink(j0, a0);
                if (v1) sink(j1, a1);
            }
        }
    };
    // candidates in LDS: keep those whose a() is within 2 delta of the n_probes-th smallest a() among
    // them (every cluster of the exact answer is among these), give them their exact distance
    auto refine = [&](uint32_t n_cand) -> uint32_t {
        const uint32_t kk = (uint32_t)n_probes < n_cand ? (uint32_t)n_probes : n_cand;
        if (kk == 0) return n_cand;
        const uint32_t limit = widen(block_kth_bound<OrderedKey>(s, n_cand, kk, [&](uint32_t i) { return t.cand_key[i]; }));
        __syncthreads();
        if (tid == 0) s.n_rec = 0;
        __syncthreads();
        // the short list, as indices into the candidate arrays (the record array is free at this point)
        for (uint32_t i = tid; i < n_cand; i += nth) {
            if (t.cand_key[i] <= limit) s.rec_pos[atomicAdd(&s.n_rec, 1u)] = i;
            else t.cand_key[i] = 0xFFFFFFFFu;
        }
        __syncthreads();
        const uint32_t n_short = s.n_rec;
        exact_all(n_short, [&](uint32_t j) { return t.cand_pos[s.rec_pos[j]]; },
                  [&](uint32_t j, float dist) { t.cand_key[s.rec_pos[j]] = __float_as_uint(dist); });
        __syncthreads();
        if (n_short > kFewMax) return n_cand;        // the others keep the all-ones key and are never selected
        // few enough for the counting selection: move the short list to the front
        const uint32_t i = (uint32_t)tid < n_short ? s.rec_pos[tid] : 0u;
        const uint32_t mk = t.cand_key[i], mp = t.cand_pos[i];
        __syncthreads();
        if ((uint32_t)tid < n_short) { t.cand_key[tid] = mk; t.cand_pos[tid] = mp; }
        __syncthreads();
        return n_short;
    };
    // compaction failed (a plateau of equal ranking values): exact distances of all clusters
    auto whole_row = [&]() -> int {
        __syncthreads();
        for (uint32_t base = 0; base < (uint32_t)n_lists; base += nth / 8) {
            const uint32_t l = base + (tid >> 3);
            const bool valid = l < (uint32_t)n_lists;
            const float dist = exact8(valid ? l : 0u, valid);
            if (valid && (tid & 7) == 0) row[l] = __float_as_uint(dist);
        }
        __threadfence_block();
        __syncthreads();
        return block_select_smallest(s, (uint32_t)n_lists, (uint32_t)n_probes,
            [&](uint32_t i) { return row[i]; }, [&](uint32_t i) { return (long long)i; });
    };
    int got;
    if constexpr (EXACT) {
        got = block_select_row(t, row, (uint32_t)n_lists, (uint32_t)n_probes, false, 0u, [](uint32_t i) { return i; },
                               [](uint32_t pos, uint32_t) { return (long long)pos; });
    } else if (S) {
        const uint32_t n_strips = ((uint32_t)n_lists + strip_w - 1) / strip_w, sw = (uint32_t)strip_w;
        const size_t stride = gridDim.x;
        const StripSummary* mine = S + q;
        // the strip minima are read several times: from the (still unused) candidate-key array if they fit; the
        // second and third keys are needed only for the few strips whose minimum passes the bound
        const bool in_lds = n_strips <= (uint32_t)CAND_CAP;         // (put there at the start; a barrier has passed)
        auto low1 = [&](uint32_t i) { return in_lds ? t.cand_key[i] : mine[i * stride].x; };
        auto low2 = [&](uint32_t i) { return mine[i * stride].y; };
        auto low3 = [&](uint32_t i) { return mine[i * stride].z; };
        const uint32_t kk = (uint32_t)n_probes < n_strips ? (uint32_t)n_probes : n_strips;
        // kk strips hold a key not above this, so it bounds the kk-th smallest key of the row
        const uint32_t bound = widen(block_kth_bound<OrderedKey>(s, n_strips, kk, [&](uint32_t i) { return low1(i) | 63u; }));
        __syncthreads();
        if (tid == 0) t.n_cand = 0;
        __syncthreads();
        for (uint32_t i = tid; i < n_strips; i += nth) {
            const uint32_t a1 = low1(i), first = i * sw;
            if ((a1 & ~63u) > bound) continue;
            const uint32_t a2 = low2(i);
            if ((a2 & ~63u) > bound || (low3(i) & ~63u) > bound) {
                // only its best cluster can pass, or its best two
                const uint32_t n_take = (a2 & ~63u) > bound ? 1u : 2u;
                for (uint32_t u = 0; u < n_take; ++u) {
                    const uint32_t c = first + ((u == 0 ? a1 : a2) & 63u);
                    if (c < (uint32_t)n_lists) {
                        const uint32_t slot = atomicAdd(&t.n_cand, 1u);
                        if (slot < (uint32_t)CAND_CAP) t.cand_pos[slot] = c;
                    }
                }
            } else {                                   // more may: all its clusters
                const uint32_t cnt = (uint32_t)n_lists - first < sw ? (uint32_t)n_lists - first : sw;
                const uint32_t slot = atomicAdd(&t.n_cand, cnt);
                for (uint32_t c = 0; c < cnt; ++c)
                    if (slot + c < (uint32_t)CAND_CAP) t.cand_pos[slot + c] = first + c;
            }
        }
        __syncthreads();
        const uint32_t n_cand = t.n_cand;
        if (n_cand >= (uint32_t)n_probes && n_cand <= (uint32_t)CAND_CAP) {
            exact_all(n_cand, [&](uint32_t j) { return t.cand_pos[j]; }, [&](uint32_t j, float dist) { t.cand_key[j] = __float_as_uint(dist); });
            __syncthreads();
            auto key_of = [&](uint32_t i) { return t.cand_key[i]; };
            auto tie_of = [&](uint32_t i) { return (long long)t.cand_pos[i]; };
            got = n_cand <= kFewMax ? block_select_few(s, n_cand, (uint32_t)n_probes, key_of, tie_of)
                                    : block_select_smallest(s, n_cand, (uint32_t)n_probes, key_of, tie_of);
            for (int j = tid; j < got; j += nth) s.rec_pos[j] = t.cand_pos[s.rec_pos[j]];
        } else {
            got = whole_row();       // a plateau of equal ranking values (or not-a-number keys)
        }
        __syncthreads();
    } else if constexpr (CAP == SEL_CAP) {
        got = block_select_row_ex<OrderedKey>(t, row, (uint32_t)n_lists, (uint32_t)n_probes, false, 0u,
                                  [](uint32_t i) { return i; },
                                  [](uint32_t pos, uint32_t) { return (long long)pos; },
                                  widen, refine, whole_row);
    } else {
        return;              // not launched: the host gives the small capacity strip summaries
    }
    if (!roff) {             // the caller's probe lists: nearest first
        for (int p = tid; p < got; p += nth) {
            probes[(size_t)q * n_probes + p] = s.rec_pos[p];
            if (probe_dists) probe_dists[(size_t)q * n_probes + p] = __uint_as_float(s.rec_key[p]);
        }
        return;
    }
    // The search's own lists.  Slot 0 is the cluster that is scanned unfiltered and whose k-th smallest R
    // bounds the rest: the nearest one that holds at least k_hint vectors (a smaller one gives no bound, and
    // then every vector of every other probe would be kept); the others follow in order of distance.
    // (lengths and first groups of all probes are fetched in parallel; got <= 1024 = the candidate buffer)
    for (int p = tid; p < got; p += nth) {
        const uint32_t l = s.rec_pos[p];
        t.cand_key[p] = list_sizes[l];
        t.cand_pos[p] = (uint32_t)group_offsets[l];
    }
    uint32_t* slot_of = reinterpret_cast<uint32_t*>(s.rec_tie);          // 2 CAP words: slot of probe p, then offsets
    uint32_t* offs = slot_of + CAP;
    __syncthreads();
    if (tid < kWave) {                     // the first wave: the pivot, then a running sum of the padded lengths in slot order
        int pivot = got;
        if (k_hint > 0)
            for (int p0 = 0; p0 < got && pivot == got; p0 += kWave) {
                const unsigned long long m = ballot64(p0 + tid < got && t.cand_key[p0 + tid < got ? p0 + tid : 0] >= (uint32_t)k_hint);
                if (m != 0) pivot = p0 + __ffsll((long long)m) - 1;
            }
        if (pivot == got) pivot = 0;
        uint32_t at = 0;
        for (int i0 = 0; i0 < got; i0 += kWave) {
            const int i = i0 + tid, p = i == 0 ? pivot : (i <= pivot ? i - 1 : i);
            const uint32_t len = i < got ? (t.cand_key[p] + 63u) & ~63u : 0u, upto = wave_inclusive_scan(len);
            if (i < got) { slot_of[p] = (uint32_t)i; offs[p] = at + upto - len; }
            at += (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
        }
        if (tid == 0) roff[(size_t)q * (n_probes + 1) + got] = at;
    }
    __syncthreads();
    for (int p = tid; p < got; p += nth) {
        const uint32_t i = slot_of[p], l = s.rec_pos[p], at = offs[p];
        probes[(size_t)q * n_probes + i] = l;
        if (probe_dists) probe_dists[(size_t)q * n_probes + i] = __uint_as_float(s.rec_key[p]);
        roff[(size_t)q * (n_probes + 1) + i] = at;
        pairs[(size_t)q * n_probes + i] = make_uint4(l, t.cand_key[p], t.cand_pos[p], at);
        if (nearest && i == 0u) nearest[q] = l;
    }
}

// One workgroup per query; the small record capacity (more workgroups per compute unit) when the selection works
// from strip summaries and n_probes allows.  Few queries leave most of the chip idle: their workgroups take 1024 threads
// (search of 1 / 16 / 512 queries, selection and top-k: 40.4 / 68.6 / 173.7 -> 38.0 / 66.5 / 172.4 us; 1024 queries
// 276 -> 287 us, hence the line at 512).
constexpr int kFewQueries = 512;

// Few queries: step 1a as the exact distances, for which the selection needs neither an error bound nor a short list.  The
// same sum as exact8 above: a group of 8 adjacent lanes per cluster, each lane every 8th component, three exchange steps; a
// group keeps the sums of QT queries, whose components wait in the LDS.
constexpr int kDirectClusters = 32;                     // per workgroup of 256 threads
template <int QT>
__global__ void __launch_bounds__(8 * kDirectClusters)
cluster_distance_kernel(const float* __restrict__ queries, const float* __restrict__ centroids, int nq, int n_lists, int d,
                        uint32_t* __restrict__ A) {
    constexpr int CH = 128;                             // components of the queries in the LDS at a time
    __shared__ float qs[CH][QT];
    const int tid = threadIdx.x, l = blockIdx.x * kDirectClusters + (tid >> 3), q0 = blockIdx.y * QT;
    const float* c = centroids + (size_t)(l < n_lists ? l : n_lists - 1) * d;
    float acc[QT];
#pragma unroll
    for (int j = 0; j < QT; ++j) acc[j] = 0.f;
    for (int k0 = 0; k0 < d; k0 += CH) {
        const int n = d - k0 < CH ? d - k0 : CH;
        float x[CH / 8];
#pragma unroll
        for (int i = 0; i < CH / 8; ++i) {
            const int u = (tid & 7) + 8 * i;
            x[i] = u < n ? c[k0 + u] : 0.f;
        }
        if (k0 > 0) __syncthreads();
        for (int i = tid; i < CH * QT; i += 8 * kDirectClusters) {
            const int j = i / CH, u = i % CH, q = q0 + j < nq ? q0 + j : nq - 1;
            qs[u][j] = u < n ? queries[(size_t)q * d + k0 + u] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < CH / 8; ++i) {
            const int u = (tid & 7) + 8 * i;           // past the last component both sides are 0, which adds nothing
            if (8 * i < n)
#pragma unroll
                for (int j = 0; j < QT; ++j) { const float diff = qs[u][j] - x[i]; acc[j] = __builtin_fmaf(diff, diff, acc[j]); }
        }
    }
#pragma unroll
    for (int j = 0; j < QT; ++j) {
        const float dist = sum_over_8_lanes(acc[j]);
        if ((tid & 7) == 0 && l < n_lists && q0 + j < nq) A[(size_t)(q0 + j) * n_lists + l] = __float_as_uint(dist);
    }
}
// Where the distances take less than the ranking values and the short list they need.  Both kernels of the probe stage, 20 probes, us,
// ranked / two queries a group / eight:
//   128 components   1,024 clusters: 1 query 12.4 / 8.3 / 8.2, 64 14.7 / 10.2 / 11.2, 130 14.8 / 12.1 / 11.2, 512 22.3 / 19.9 / 16.1
//                    3,000: 16 queries 14.6 / 10.1 / 11.3, 64 15.6 / 13.0 / 11.5, 130 14.8 / 16.7 / 14.2, 256 15.5 / - / 17.6
//                    8,000: 1 query 12.5 / 10.7 / 10.9, 16 13.3 / 13.1 / 12.9, 64 13.3 / 20.7 / 16.9
//   512 components   1,024: 1 query 25.7 / 11.9, 64 28.1 / 15.8 / 19.0, 512 39.1 / 45.2 / 30.4; 8,000: 16 queries 31.1 / 24.7 / 22.3
// (Of many clusters the selection reads strip summaries, a thirtieth of the distances.)
bool direct_distances(int nq, int n_lists) {
    return nq <= kFewQueries && (n_lists <= 1024 || (n_lists <= 8192 && (size_t)nq * n_lists <= (size_t)3 << 16));
}
// Step 1a for nq queries: exact distances or ranking keys in A, or strip summaries in S (null on return: not made).
int launch_step_1a(const ivfpq_index* idx, const float* q, int nq, int n_probes, uint32_t* A, StripSummary** S, bool* exact, void* split_ws, hipStream_t st) {
    const int n_lists = idx->n_lists, d = idx->d;
    *exact = direct_distances(nq, n_lists);
    if (*exact || !coarse_use_strips(nq, n_lists, n_probes)) *S = nullptr;
    if (!*exact) return launch_coarse(q, idx->dev.centroids, idx->dev.centroid_norms, nq, n_lists, d, A, *S, split_ws, st);
    const float* centroids = idx->dev.centroids;
    const unsigned blocks = (unsigned)((n_lists + kDirectClusters - 1) / kDirectClusters);
    auto go = [&](auto kernel, int qt) {
        hipLaunchKernelGGL(kernel, dim3(blocks, (unsigned)((nq + qt - 1) / qt)), dim3(8 * kDirectClusters), 0, st, q, centroids, nq, n_lists, d, A);
    };
    if ((size_t)nq * n_lists <= (size_t)1 << 16) go(cluster_distance_kernel<2>, 2);       // (the figures above)
    else go(cluster_distance_kernel<8>, 8);
    HIP_TRY(hipGetLastError());
    return IVFPQ_OK;
}

void launch_select_probes(int nq, bool exact, hipStream_t st, uint32_t* A, const StripSummary* S, int strip_w, const float* queries,
                          const float* centroids, float centroid_norm_max, const ivfpq::RankCrowd& crowd, int d, int n_lists, int n_probes, const uint32_t* list_sizes,
                          const int64_t* group_offsets, uint32_t* probes, float* probe_dists, uint32_t* roff, uint4* pairs, int k_hint, uint32_t* nearest = nullptr) {
    if (!exact && !S && select_by_waves(nq, n_probes, crowd.of(n_probes))) {
        hipLaunchKernelGGL(select_probes_wave_kernel, dim3((unsigned)((nq + kWaveQueries - 1) / kWaveQueries)), dim3(64 * kWaveQueries), 0, st, A, queries, centroids,
                           centroid_norm_max, d, n_lists, n_probes, nq, list_sizes, group_offsets, probes, probe_dists, roff, pairs, k_hint, nearest);
        return;
    }
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(nq), dim3(threads), 0, st, A, S, strip_w, queries, centroids, centroid_norm_max, d, n_lists, n_probes, list_sizes, group_offsets,
                           probes, probe_dists, roff, pairs, k_hint, nearest);
    };
    if (exact) go(select_probes_kernel<SEL_CAP, 1024, true>, 1024);
    else if (nq <= kFewQueries) go(select_probes_kernel<SEL_CAP, 1024>, 1024);
    else if (S && n_probes <= SEL_CAP_SMALL) go(select_probes_kernel<SEL_CAP_SMALL, SEL_THREADS>, SEL_THREADS);
    else go(select_probes_kernel<SEL_CAP, SEL_THREADS>, SEL_THREADS);
}

// Same layout step for caller-given probes.
__global__ void __launch_bounds__(256)
layout_probes_kernel(const uint32_t* __restrict__ probes_in, int nq, int n_probes, int n_lists,
                     const uint32_t* __restrict__ list_sizes, const int64_t* __restrict__ group_offsets,
                     uint32_t* __restrict__ probes, uint32_t* __restrict__ roff, uint4* __restrict__ pairs) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    uint32_t at = 0;
    for (int p = 0; p < n_probes; ++p) {
        uint32_t l = probes_in[(size_t)q * n_probes + p];
        const bool ok = l < (uint32_t)n_lists;                 // an out-of-range entry is skipped
        const uint32_t len = ok ? list_sizes[l] : 0u;
        probes[(size_t)q * n_probes + p] = l;
        roff[(size_t)q * (n_probes + 1) + p] = at;
        pairs[(size_t)q * n_probes + p] = make_uint4(l, len, ok ? (uint32_t)group_offsets[l] : 0u, at);
        at += (len + 63u) & ~63u;
    }
    roff[(size_t)q * (n_probes + 1) + n_probes] = at;
}

// ================================================================================================
// Steps 2-4: residual, lookup table in LDS, code scan.
// ================================================================================================
template <int LUT>
__device__ inline void store4(unsigned char* lut, int e, const float f[4], const Fp8Params fp8, int hi_v) {
    if constexpr (LUT == IVFPQ_LUT_FP32) {
        *reinterpret_cast<float4*>(lut + (size_t)e * 4) = make_float4(f[0], f[1], f[2], f[3]);
    } else if constexpr (LUT == IVFPQ_LUT_FP16) {
        uint2 v;
        v.x = half_bits_from_f32(f[0]) | (half_bits_from_f32(f[1]) << 16);
        v.y = half_bits_from_f32(f[2]) | (half_bits_from_f32(f[3]) << 16);
        *reinterpret_cast<uint2*>(lut + (size_t)e * 2) = v;
    } else {
        constexpr int SH = Fp8Format<LUT>::shift;
        *reinterpret_cast<uint32_t*>(lut + e) = fp8_pack4<SH>(f, fp8, hi_v);
    }
}

// Visits every entry of F[pq_dim][ksub], 4 consecutive entries of one sub-space per call of
// sink(first entry index, values) (ksub is 16 or 256, so 4 consecutive entries never straddle
// sub-spaces).  codebooks: global [pq_dim][ksub][M]; rq: LDS [pq_dim*M].
template <int M, class Sink>
__device__ __forceinline__ void visit_lut(const float* __restrict__ codebooks, const float* rq, int e_begin, int n_entries,
                                 int bits, int m_runtime, Sink sink) {
    for (int e = e_begin + threadIdx.x * 4; e < n_entries; e += blockDim.x * 4) {
        const int j = e >> bits;
        float f[4];
        if constexpr (M > 0) {
            float r[M];
#pragma unroll
            for (int t = 0; t < M; ++t) r[t] = rq[j * M + t];
            float cbv[4 * M];
            const float4* src = reinterpret_cast<const float4*>(codebooks + (size_t)e * M);
#pragma unroll
            for (int v = 0; v < M; ++v) {
                float4 x = src[v];
                cbv[4 * v] = x.x; cbv[4 * v + 1] = x.y; cbv[4 * v + 2] = x.z; cbv[4 * v + 3] = x.w;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) f[u] = lut_entry<M>(cbv + u * M, r);
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float* cbv = codebooks + (size_t)(e + u) * m_runtime;
                float acc = 0.f;
                for (int t = 0; t < m_runtime; ++t) {
                    float diff = cbv[t] - rq[j * m_runtime + t];
                    acc = __builtin_fmaf(diff, diff, acc);
                }
                f[u] = acc;
            }
        }
        sink(e, f);
    }
}

// 8-bit codes: a table row has 256 entries = 4 per lane of a wave, so every wave visits whole rows
// (row index wave-uniform: residual components are read once per row, addresses advance by a
// constant stride).
template <int M, class Sink>
__device__ __forceinline__ void visit_lut_rows256(const float* __restrict__ codebooks, const float* rq, int row0, int pq_dim, Sink sink) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_waves = blockDim.x >> 6;
    const size_t src_step = (size_t)n_waves * 256 * M;
    const int e_step = n_waves * 256;
    auto load_row = [&](const float* src, float (&cbv)[4 * M]) {
#pragma unroll
        for (int v = 0; v < M; ++v) {
            float4 x = reinterpret_cast<const float4*>(src)[v];
            cbv[4 * v] = x.x; cbv[4 * v + 1] = x.y; cbv[4 * v + 2] = x.z; cbv[4 * v + 3] = x.w;
        }
    };
    auto finish_row = [&](const float (&cbv)[4 * M], int j, int e) {
        float r[M];
#pragma unroll
        for (int t = 0; t < M; ++t) r[t] = rq[j * M + t];
        float f[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) f[u] = lut_entry<M>(cbv + u * M, r);
        sink(e, f);
    };
    const float* src = codebooks + ((size_t)(row0 + wave) * 256 + lane * 4) * M;
    int e = (row0 + wave) * 256 + lane * 4;
    int j = row0 + wave;
    // two rows per trip (written out: both rows' loads are in flight before either is used; deeper
    // prefetching costs registers, hence occupancy, and measured slower)
    for (; j + n_waves < pq_dim; j += 2 * n_waves) {
        float c0[4 * M], c1[4 * M];
        load_row(src, c0);
        load_row(src + src_step, c1);
        finish_row(c0, j, e);
        finish_row(c1, j + n_waves, e + e_step);
        src += 2 * src_step;
        e += 2 * e_step;
    }
    if (j < pq_dim) {
        float c0[4 * M];
        load_row(src, c0);
        finish_row(c0, j, e);
    }
}

// rows (sub-spaces) row0 .. row1 - 1 of the table
template <int BITS, class Sink>
__device__ __forceinline__ void visit_lut_any_m(const float* __restrict__ codebooks, const float* rq, int row0, int row1, int m, Sink sink) {
    const int e_begin = row0 << BITS, e_end = row1 << BITS;
    if constexpr (BITS == 8) {
        switch (m) {
            case 1: visit_lut_rows256<1>(codebooks, rq, row0, row1, sink); return;
            case 2: visit_lut_rows256<2>(codebooks, rq, row0, row1, sink); return;
            case 4: visit_lut_rows256<4>(codebooks, rq, row0, row1, sink); return;
            default: break;
        }
    }
    switch (m) {
        case 1: visit_lut<1>(codebooks, rq, e_begin, e_end, BITS, m, sink); break;
        case 2: visit_lut<2>(codebooks, rq, e_begin, e_end, BITS, m, sink); break;
        case 4: visit_lut<4>(codebooks, rq, e_begin, e_end, BITS, m, sink); break;
        default: visit_lut<0>(codebooks, rq, e_begin, e_end, BITS, m, sink); break;
    }
}

// Step 3: builds F[pq_dim][ksub] in LDS in the table's dtype; rq must be complete (barrier passed).
// Ends with a barrier.  Returns the constants the 8-bit lookups decode with (workgroup-uniform).
// Per-table bias (a power-of-two scale of the table, expressed as a shift of the format's exponent
// bias): a first pass over the entries finds the largest one; with e its FP32 exponent, the bias is
// top_exp - e, so that the entry's binade becomes the format's top binade; a second pass encodes.
// row0, row1: only these rows (sub-spaces) are built (the whole table for a per-table bias, which needs its
// largest entry).
template <int LUT, int BITS>
__device__ __forceinline__ Fp8Params stage_table(const float* __restrict__ codebooks, const float* rq, int pq_dim, int m,
                                        unsigned char* lut, uint32_t* max_slot, const Fp8Mode mode, int row0, int row1) {
    Fp8Params fp8 = mode.fixed;
    if constexpr (kIsFp8<LUT>) {
        if (mode.per_table) {
            if (threadIdx.x == 0) *max_slot = 0u;
            __syncthreads();
            float mx = 0.f;                       // entries are sums of squares: never negative
            row0 = 0; row1 = pq_dim;
            visit_lut_any_m<BITS>(codebooks, rq, 0, pq_dim, m, [&](int, const float (&f)[4]) {
                mx = fmaxf(fmaxf(mx, f[0]), fmaxf(f[1], fmaxf(f[2], f[3])));
            });
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
            if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(max_slot, __float_as_uint(mx));
            __syncthreads();
            const int e = (int)(*max_slot >> 23) - 127;
            int bias = Fp8Format<LUT>::top_exp - e;
            bias = min(max(bias, Fp8Format<LUT>::bias_min), Fp8Format<LUT>::bias_max);
            bias = __builtin_amdgcn_readfirstlane(bias);
            fp8 = fp8_params(Fp8Format<LUT>::shift, bias, mode.truncate);
        }
    }
    int hi_v = fp8.hi;
    asm volatile("" : "+v"(hi_v));       // the upper clamp limit, held in a vector register
    visit_lut_any_m<BITS>(codebooks, rq, row0, row1, m, [&](int e, const float (&f)[4]) { store4<LUT>(lut, e, f, fp8, hi_v); });
    __syncthreads();
    return fp8;
}

template <int LUT>
__device__ inline float lut_get(const unsigned char* lut, uint32_t idx, const Fp8Params fp8) {
    if constexpr (LUT == IVFPQ_LUT_FP32) return reinterpret_cast<const float*>(lut)[idx];
    else if constexpr (LUT == IVFPQ_LUT_FP16) return __half2float(reinterpret_cast<const __half*>(lut)[idx]);
    else return fp8_to_f32<Fp8Format<LUT>::shift>(lut[idx], fp8);
}

// Bit-packed codes: the codes of a vector are one bit string, sub-space j in bits [j*BITS, (j+1)*BITS).
// A "code group" is the shortest run of sub-spaces that ends on a 32-bit boundary: SPG sub-spaces in
// WPG words (8 in 1 for 4-bit codes, 4 in 1 for 8-bit, 32 in 5 / 16 in 3 / 32 in 7 for 5 / 6 / 7 bits).
template <int BITS> struct CodeGroup {
    static constexpr int g = (BITS % 8 == 0) ? 8 : (BITS % 4 == 0) ? 4 : (BITS % 2 == 0) ? 2 : 1;   // gcd(BITS, 32)
    static constexpr int SPG = 32 / g, WPG = BITS / g;
};

// adds the table entries selected by the SPG codes held in w[0 .. WPG) (sub-spaces row0.. ascending)
template <int LUT, int BITS>
__device__ inline float add_group(float acc, const unsigned char* lut, const uint32_t* w, int row0, const Fp8Params fp8) {
    constexpr int SPG = CodeGroup<BITS>::SPG, KSUB = 1 << BITS;
    if constexpr (BITS == 8 && (LUT == IVFPQ_LUT_FP16 || LUT == IVFPQ_LUT_FP32)) {
        // Whole-byte codes and entries of 2 or 4 bytes: the entry's byte offset in its row comes out of one
        // sub-dword shift, the row's offset goes into the LDS read's immediate, and a half entry is converted by
        // the instruction that adds it: 2 vector instructions per lookup.  (The table sits at LDS address 0: the
        // kernel has no static LDS, which the host verifies before the first launch.)
        constexpr int E = LutTraits<LUT>::bytes, LG = ilog2(E);
        const uint32_t off[4] = {byte_shl<0, LG>(w[0]), byte_shl<1, LG>(w[0]), byte_shl<2, LG>(w[0]), byte_shl<3, LG>(w[0])};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const uint32_t x = LdsWord<E>::load(off[s] + (uint32_t)(row0 + s) * (uint32_t)(KSUB * E));
            if constexpr (LUT == IVFPQ_LUT_FP16) acc = add_half_lo(acc, x);
            else acc += __uint_as_float(x);
        }
        return acc;
    }
    if constexpr (BITS == 4 && (LUT == IVFPQ_LUT_FP16 || LUT == IVFPQ_LUT_FP32)) {
        // The same for nibbles, eight of them after two masks (as in the group kernel), the eight reads before the first add.  Nearest-probe
        // scan of 10,000 queries, 64 sub-spaces, half tables, lists of 2,000: 354 -> 273 us.  (One-byte and bit-packed
        // entries gain nothing from reads taken together: 178 -> 185 us with 7 bits.)
        constexpr int E = LutTraits<LUT>::bytes, LG = ilog2(E);
        constexpr uint32_t kNibbles = 0x0F0F0F0Fu << LG;
        const uint32_t lo4 = (w[0] << LG) & kNibbles, hi4 = (w[0] >> (4 - LG)) & kNibbles;
        const uint32_t off[8] = {byte_shl<0, 0>(lo4), byte_shl<0, 0>(hi4), byte_shl<1, 0>(lo4), byte_shl<1, 0>(hi4),
                                 byte_shl<2, 0>(lo4), byte_shl<2, 0>(hi4), byte_shl<3, 0>(lo4), byte_shl<3, 0>(hi4)};
        uint32_t x[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) x[s] = LdsWord<E>::load(off[s] + (uint32_t)(row0 + s) * (uint32_t)(KSUB * E));
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if constexpr (LUT == IVFPQ_LUT_FP16) acc = add_half_lo(acc, x[s]);
            else acc += __uint_as_float(x[s]);
        }
        return acc;
    }
#pragma unroll
    for (int s = 0; s < SPG; ++s) {
        constexpr uint32_t mask = (uint32_t)KSUB - 1u;
        const int bit = s * BITS, wi = bit >> 5, sh = bit & 31;
        uint32_t code;
        if (sh + BITS <= 32) code = (w[wi] >> sh) & mask;
        else code = ((w[wi] >> sh) | (w[wi + 1] << (32 - sh))) & mask;     // the field straddles two words
        acc += lut_get<LUT>(lut, (uint32_t)(row0 + s) * (uint32_t)KSUB + code, fp8);
    }
    return acc;
}

constexpr int kBoundBins = 1024;
constexpr size_t kBoundLds = (size_t)kBoundBins * 4 + 64;

// The end of a workgroup that has written all R of its query's nearest probe (row[0 .. len)): an upper bound of the k-th
// smallest of them, hence of the query's k-th smallest R, for the scan of the other probes, and the values not above it as
// the first entries of the query's survivor list (behind the segment: value and position).  Fewer than k finite values: no bound, every
// vector is admitted.
// The bound is the upper edge of the histogram bin that holds the k-th smallest: 1,024 equal bins between the least and the
// largest value, and again inside the bin where it holds many (values that cluster).  A few values past the k-th may be listed; the
// selection at the end is exact.  (A kernel of its own that selected the k-th exactly, four rounds of digits with a dozen barriers, took 72 us
// after the 153 us of the scan, 10,000 queries on 10^6 vectors.)
// lo, hi: least and largest finite value this lane has written (bits; all-ones and 0 if none).
__device__ __forceinline__ void bound_of_nearest(const ScanArgs& a, int q, uint32_t len, unsigned char* smem, uint32_t lo, uint32_t hi) {
    uint32_t* hist = reinterpret_cast<uint32_t*>(smem);
    uint32_t* box = hist + kBoundBins;                       // least, largest, bin, values below it, values in it, listed
    const int tid = threadIdx.x, nth = blockDim.x, lane = tid & (kWave - 1);
    // the counters of the grouping that follows
#pragma unroll
    for (int c = 0; c < 2; ++c)
        for (uint32_t i = (uint32_t)q * nth + tid; i < a.n_clear[c]; i += gridDim.x * nth) a.clear[c][i] = 0u;
    const uint32_t seg0 = (len + 63u) & ~63u, k = (uint32_t)a.k_bound;
    uint32_t* row = reinterpret_cast<uint32_t*>(a.R + (size_t)q * a.stride);
    uint32_t* row_pos = a.Rpos + (size_t)q * a.stride;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off, kWave));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off, kWave));
    }
    __syncthreads();                                         // the tables are done with, the values in place
    if (tid < 6) box[tid] = tid == 0 ? 0xFFFFFFFFu : 0u;
    for (int b = tid; b < kBoundBins; b += nth) hist[b] = 0u;
    __syncthreads();
    if (lane == 0) { atomicMin(&box[0], lo); atomicMax(&box[1], hi); }
    __syncthreads();
    float from = __uint_as_float(box[0]), to = __uint_as_float(box[1]);
    const bool any = box[0] <= box[1];
    // sink(key, position) of every value: where a thread has several, four are read before the first is used, since one read after the
    // other waits for memory each time (nearest-probe scan of 10,000 queries, lists of 1,000 / 2,000: 190 -> 179 / 394 -> 361 us)
    auto each_key = [&](auto sink) __attribute__((always_inline)) {
        uint32_t base = 0;
        for (; base + 4u * nth <= len; base += 4u * nth) {
            uint32_t v[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) v[u] = row[base + u * nth + tid];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) sink(v[u], base + u * nth + tid);
        }
        for (; base < len; base += nth) sink(base + tid < len ? row[base + tid] : kPadKey, base + tid);
    };
    uint32_t bound = kAdmitAll, below = 0;                   // below: values less than `from`
    for (int round = 0; any && len >= k && round < 4; ++round) {
        const float width = (to - from) * (1.f / (kBoundBins - 1)), inv = width > 0.f ? 1.f / width : 0.f;
        each_key([&](uint32_t key, uint32_t) {
            const float v = __uint_as_float(key);
            if (key < 0x7F800000u && v >= from && v <= to) {
                const int b = (int)((v - from) * inv);
                atomicAdd(&hist[b < kBoundBins - 1 ? b : kBoundBins - 1], 1u);
            }
        });
        __syncthreads();
        if (tid < kWave) {
            uint32_t c[kBoundBins / kWave], sum = 0;
#pragma unroll
            for (int u = 0; u < kBoundBins / kWave; ++u) { c[u] = hist[tid * (kBoundBins / kWave) + u]; sum += c[u]; }
            uint32_t at = below + wave_inclusive_scan(sum) - sum;
            if (tid == 0) box[2] = 0xFFFFFFFFu;
#pragma unroll
            for (int u = 0; u < kBoundBins / kWave; ++u) {
                if (at < k && k <= at + c[u]) { box[2] = (uint32_t)(tid * (kBoundBins / kWave) + u); box[3] = at; box[4] = c[u]; }
                at += c[u];
            }
        }
        __syncthreads();
        const uint32_t bin = box[2], before = box[3], in_bin = box[4];
        if (bin == 0xFFFFFFFFu) break;                       // fewer than k finite values
        // everything counted up to this bin is at most its edge: the roundings of the bin's number and of the edge are within 2^-21
        // (of subnormal values a bin's width is rounded to few bits or to none: the last bin, which takes all above it, and the
        // only one where there is no width, end at the largest value)
        const float edge = width > 0.f && bin < (uint32_t)kBoundBins - 1u ? fminf((from + (float)(bin + 1) * width * 1.000001f) * 1.0000005f, to) : to;
        bound = __float_as_uint(edge);
        if (before + in_bin <= k + k / 8 + 8 || width * 1048576.f <= to) break;
        const float start = fmaxf(from, (from + (float)bin * width * 0.999999f) * 0.9999995f);
        // again inside the bin (its edges taken a little wide: what lies between is counted as below only if it was)
        __syncthreads();
        for (int b = tid; b < kBoundBins; b += nth) hist[b] = 0u;
        if (tid == 0) box[2] = 0u;
        __syncthreads();
        uint32_t less = 0;
        for (uint32_t i = tid; i < len; i += nth) {
            const uint32_t key = row[i];
            less += key < 0x7F800000u && __uint_as_float(key) < start ? 1u : 0u;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) less += (uint32_t)__shfl_xor((int)less, off, kWave);
        if (lane == 0) atomicAdd(&box[2], less);
        __syncthreads();
        below = box[2];
        from = start;
        to = edge;
        __syncthreads();
    }
    each_key([&](uint32_t key, uint32_t i) {
        const unsigned long long m = ballot64(key <= bound);
        if (m == 0) return;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&box[5], (uint32_t)__popcll(m));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + lanes_below(m);
        if (key <= bound) { row[seg0 + at] = key; row_pos[seg0 + at] = i; }
    });
    __syncthreads();
    if (tid == 0) {
        a.bounds[q] = bound;
        a.counts[q] = box[5];
        if (a.starts) a.starts[q] = box[5];
    }
}

constexpr int kStageCap = 128;   // survivors a wave stages in LDS before it appends them (8 bytes each)

// Code layout of one cluster (written by ivfpq_upload): vectors in groups of 64 (the last one
// zero-padded); inside a group, chunk c of all 64 vectors is contiguous:
//   byte address = ((group * n_chunks + c) * 64 + lane) * CW
// so one wave-wide load of chunk c reads 64*CW contiguous bytes.
template <int LUT, int BITS, int CW, int NCH>
__global__ void __launch_bounds__(1024)
scan_kernel(ScanArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int ksub = 1 << BITS;
    const int n_entries = a.pq_dim * ksub;
    // LDS: table | residual (d floats) | 16 bytes (largest entry, per-table bias) | survivor staging
    unsigned char* lut = smem;
    float* rq = reinterpret_cast<float*>(smem + (((size_t)n_entries * LutTraits<LUT>::bytes + 15) & ~(size_t)15));
    unsigned char* after_rq = reinterpret_cast<unsigned char*>(rq) + (((size_t)a.d * 4 + 15) & ~(size_t)15);
    uint32_t* max_slot = reinterpret_cast<uint32_t*>(after_rq);
    Fp8Params fp8 = a.fp8.fixed;

    int q, l;
    uint32_t len, first_group, row_pos0 = 0;
    float* Rout;
    if (a.single_list >= 0) {
        q = 0; l = a.single_list; Rout = a.R;
        len = a.list_sizes[l];
        first_group = (uint32_t)a.group_offsets[l];
    } else {
        size_t pair_idx;
        if (a.mode == 1) {
            q = blockIdx.x;
            pair_idx = (size_t)q * a.n_probes;
        } else if (a.mode == 3) {                              // all probes of a query in a row, unfiltered
            q = blockIdx.x / a.n_probes;
            pair_idx = blockIdx.x;
        } else if (a.order == nullptr) {
            q = blockIdx.x / (a.n_probes - 1);
            pair_idx = (size_t)q * a.n_probes + 1 + (blockIdx.x - q * (a.n_probes - 1));
        } else {
            // Pairs grouped by cluster, and workgroups go round-robin to the 8 XCDs: blocks of
            // `order_block` consecutive pairs of the grouped order are dealt to the XCDs in turn, so that
            // the workgroups scanning one cluster run on one XCD (a few, for a cluster with many pairs)
            // at about the same time and its codes come from that XCD's L2 after the first read.
            const uint32_t xcd = blockIdx.x & 7u, rank = blockIdx.x >> 3;
            const uint32_t slot = ((rank / a.order_block) * 8u + xcd) * a.order_block + rank % a.order_block;
            if (slot >= a.n_pairs) return;
            const uint32_t lin = a.order[slot];
            q = (int)(lin / (uint32_t)(a.n_probes - 1));
            pair_idx = (size_t)q * a.n_probes + 1 + (lin - (uint32_t)q * (uint32_t)(a.n_probes - 1));
        }
        const uint4 pair = a.pairs[pair_idx];
        l = (int)pair.x; len = pair.y; first_group = pair.z;
        Rout = a.R + (size_t)q * a.stride + pair.w;
        row_pos0 = pair.w;
    }
    const bool bounded = a.single_list < 0 && a.mode == 1 && a.k_bound > 0;
    // An empty cluster, or a caller-given probe that was out of range, whose l names no centroid: no residual and no table, only
    // the bound (len is the same for the whole workgroup)
    if (len == 0 && !bounded) return;
    uint32_t least = 0xFFFFFFFFu, largest = 0;                     // mode 1: of the finite values this lane has written
    const bool filtered = a.single_list < 0 && a.mode == 2;
    const bool prune = filtered && a.early_exit != 0;
    uint32_t bound = 0, seg0 = 0;
    if (filtered) {
        bound = a.bounds[q];
        seg0 = a.pairs[(size_t)q * a.n_probes + 1].w;     // padded length of the nearest probe's segment
    }
    // filtered mode: every wave stages its survivors in a private LDS buffer and appends them to the
    // query's row with one global atomic per flush (the counter of a query is shared by all the
    // workgroups of that query: one atomic per 64-vector group would serialise on it)
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));    // the same for the whole wave: loop counters and group addresses stay scalar
    uint2* stage = reinterpret_cast<uint2*>(after_rq + 16) + (size_t)wave * kStageCap;
    uint32_t staged = 0;       // wave-uniform
    const int n_groups = (int)((len + 63u) >> 6);
    const int lane = threadIdx.x & (kWave - 1);
    const int n_waves = blockDim.x >> 6;
    const int nch = NCH > 0 ? NCH : a.n_chunks;
    const uint8_t* codes_l = a.codes + (size_t)first_group * 64 * ((size_t)nch * CW);

    using chunk_t = typename std::conditional<CW == 16, uint4, uint32_t>::type;
    const chunk_t* cbase = reinterpret_cast<const chunk_t*>(codes_l);

    constexpr int NBUF = NCH > 0 ? NCH : 1;
    constexpr int SPG = CodeGroup<BITS>::SPG, WPG = CodeGroup<BITS>::WPG;

    auto load_group = [&](chunk_t (&buf)[NBUF], int g) {
#pragma unroll
        for (int c = 0; c < NBUF; ++c) buf[c] = cbase[((size_t)g * NBUF + c) * 64 + lane];
    };
    // Eq. (1) for the vector this lane holds in buf: sub-spaces in ascending order
    // (blocks_tag: how many blocks of kBlockSub sub-spaces to add, the leading ones; NBLK = all)
    constexpr int NG = CW == 16 ? (4 * NBUF) / WPG : 0;                          // code groups per vector
    constexpr int EVERY = 16 / SPG > 0 ? 16 / SPG : 1;                           // code groups per block of 16 sub-spaces
    constexpr int NBLK = (NG + EVERY - 1) / EVERY;
    auto accumulate = [&](const chunk_t (&buf)[NBUF], auto blocks_tag) -> float {
        constexpr int BLOCKS = decltype(blocks_tag)::value;
        float acc = 0.f;
        if constexpr (CW == 16) {
            uint32_t w[4 * NBUF];
#pragma unroll
            for (int c = 0; c < NBUF; ++c) { w[4 * c] = buf[c].x; w[4 * c + 1] = buf[c].y; w[4 * c + 2] = buf[c].z; w[4 * c + 3] = buf[c].w; }
            static_assert((4 * NBUF) % WPG == 0 || NCH == 0, "16-byte chunks must hold whole code groups");
            // Table entries are never negative, so the partial sums only grow: once those of all 64
            // vectors are over the query's bound none of them can survive, and the rest of their
            // lookups is skipped (checked every 16 sub-spaces; the partial sum then fails the filter).
            bool over = false;                       // wave-uniform
#pragma unroll
            for (int blk = 0; blk < BLOCKS; ++blk) {
                if (over) continue;
#pragma unroll
                for (int e = 0; e < EVERY; ++e) {
                    const int cg = blk * EVERY + e;
                    if (cg < NG) acc = add_group<LUT, BITS>(acc, lut, w + cg * WPG, cg * SPG, fp8);
                }
                if (blk + 1 < BLOCKS && prune) over = ballot64(__float_as_uint(acc) <= bound) == 0;
            }
        }
        return acc;      // 4-byte chunks take the loop over code groups below instead
    };
    auto flush_stage = [&]() {
        if (staged == 0) return;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&a.counts[q], staged);
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        uint32_t* dst_key = reinterpret_cast<uint32_t*>(a.R) + (size_t)q * a.stride + seg0 + base;
        uint32_t* dst_pos = a.Rpos + (size_t)q * a.stride + seg0 + base;
        for (uint32_t j = lane; j < staged; j += kWave) {
            const uint2 e = stage[j];
            dst_key[j] = e.x;
            dst_pos[j] = e.y;
        }
        staged = 0;
    };
    auto store_R = [&](int g, float acc) {
        const uint32_t i = (uint32_t)g * 64u + lane;
        if (!filtered) {
            if (i < len) {
                Rout[i] = acc;
                const uint32_t key = __float_as_uint(acc);
                if (key < 0x7F800000u) { least = min(least, key); largest = max(largest, key); }
            } else if (a.single_list < 0) Rout[i] = __uint_as_float(kPadKey);   // padding slot of the R scratch
        } else {
            // keep only what can still be among the k best
            // (the mask is the AND of two compares' results; a ballot of their conjunction goes through a 0/1 value)
            const bool keep = i < len && __float_as_uint(acc) <= bound;
            const unsigned long long m = ballot64(i < len) & ballot64(__float_as_uint(acc) <= bound);
            if (m != 0) {
                if (staged + 64u > (uint32_t)kStageCap) flush_stage();
                if (keep) stage[staged + lanes_below(m)] = make_uint2(__float_as_uint(acc), row_pos0 + i);
                staged += (uint32_t)__popcll(m);
            }
        }
    };

    // issue the loads of this wave's first group before the table is built: HBM latency overlaps it
    chunk_t buf_a[NBUF], buf_b[NBUF];
    int g = wave;
    if constexpr (NCH > 0) {
        if (g < n_groups) load_group(buf_a, g);
    }

    // step 2: residual of the query against this cluster's centroid
    if (len != 0)
        for (int t = threadIdx.x; t < a.d; t += blockDim.x)
            rq[t] = a.queries[(size_t)q * a.d + t] - a.centroids[(size_t)l * a.d + t];
    __syncthreads();
    // Filtered scan with early exit, tables of two or more chunks' worth of rows: most groups are over the
    // bound after the first half of the sub-spaces, so the second half of the table is built only if some
    // group of this pair is still in the race.  Pass 1 builds the leading rows and adds them up for every
    // group, noting the groups with a partial sum under the bound; if there are any, the remaining rows are
    // built and those groups are added up from the start (same order: same R).
    constexpr int HBLK = (NBLK + 1) / 2;                             // blocks of the first pass
    constexpr int HROWS = HBLK * EVERY * SPG;                        // table rows they use
    constexpr int HCH = (HBLK * EVERY * WPG + 3) / 4;                // 16-byte chunks that hold their codes
    // Worth it only if the first pass weeds out most groups and the rows it saves are expensive.  Measured
    // (scan stage, 10,000 queries): 64 sub-spaces of 8-bit codes, first pass 32: 2.13 -> 1.68 ms (e5m3), 3.06 ->
    // 2.74 ms (fp32); 48 sub-spaces, first pass 32: 2.20 -> 2.47 ms (fp32); 32 sub-spaces, first pass 16: 6.5 ->
    // 8.1 ms (most groups went through twice); 4-bit codes (16-entry rows cost nothing to build): 6.8 -> 9.7 ms.
    // Hence: 8-bit codes, four chunks, the first pass takes half of them.
    constexpr bool kCanSplit = BITS == 8 && NCH == 4 && HROWS >= 32 && 2 * HBLK == NBLK;
    bool lazy = false;
    if constexpr (kCanSplit) lazy = prune && !(kIsFp8<LUT> && a.fp8.per_table);
    if constexpr (kCanSplit) {
        if (lazy) {
            uint32_t* any_alive = max_slot + 1;
            uint16_t* alive = reinterpret_cast<uint16_t*>(after_rq + 16 + (size_t)n_waves * kStageCap * 8) + (size_t)wave * kAliveCap;
            if (threadIdx.x == 0) *any_alive = 0u;
            fp8 = stage_table<LUT, BITS>(a.codebooks, rq, a.pq_dim, a.m, lut, max_slot, a.fp8, 0, HROWS);
            uint32_t n_alive = 0;                // wave-uniform
            bool redo_all = false;               // more groups in the race than the list holds: take them all again
            auto load_head = [&](chunk_t (&buf)[NBUF], int grp) {
#pragma unroll
                for (int c = 0; c < HCH; ++c) buf[c] = cbase[((size_t)grp * NBUF + c) * 64 + lane];
            };
            auto first_pass = [&](int grp, const chunk_t (&buf)[NBUF]) {
                const float acc = accumulate(buf, std::integral_constant<int, HBLK>{});
                if ((ballot64((uint32_t)grp * 64u + lane < len) & ballot64(__float_as_uint(acc) <= bound)) != 0) {
                    if (n_alive < (uint32_t)kAliveCap && grp / n_waves < 65536) { if (lane == 0) alive[n_alive] = (uint16_t)(grp / n_waves); ++n_alive; }
                    else redo_all = true;
                }
            };
            // (the loads of the wave's first group were issued in full above; later groups load the head only)
            while (g < n_groups) {
                const int gn = g + n_waves;
                if (gn < n_groups) load_head(buf_b, gn);
                first_pass(g, buf_a);
                if (gn >= n_groups) break;
                g = gn + n_waves;
                if (g < n_groups) load_head(buf_a, g);
                first_pass(gn, buf_b);
            }
            if (lane == 0 && (n_alive != 0 || redo_all)) atomicOr(any_alive, 1u);
            __syncthreads();
            if (*any_alive == 0u) return;
            (void)stage_table<LUT, BITS>(a.codebooks, rq, a.pq_dim, a.m, lut, max_slot, a.fp8, HROWS, a.pq_dim);
            if (redo_all) {
                for (g = wave; g < n_groups; g += n_waves) {
                    load_group(buf_a, g);
                    store_R(g, accumulate(buf_a, std::integral_constant<int, NBLK>{}));
                }
            } else {
                for (uint32_t t = 0; t < n_alive; ++t) {
                    g = (int)alive[t] * n_waves + wave;
                    load_group(buf_a, g);
                    store_R(g, accumulate(buf_a, std::integral_constant<int, NBLK>{}));
                }
            }
            flush_stage();
            return;
        }
    }
    // step 3: the table
    if (len != 0) fp8 = stage_table<LUT, BITS>(a.codebooks, rq, a.pq_dim, a.m, lut, max_slot, a.fp8, 0, a.pq_dim);

    // step 4: Eq. (1), one lane per coded vector; the next group is loaded into the other register
    // buffer while the current one is looked up
    if constexpr (NCH > 0) {
        while (g < n_groups) {
            int gn = g + n_waves;
            if (gn < n_groups) load_group(buf_b, gn);
            store_R(g, accumulate(buf_a, std::integral_constant<int, NBLK>{}));
            if (gn >= n_groups) break;
            g = gn + n_waves;
            if (g < n_groups) load_group(buf_a, g);
            store_R(gn, accumulate(buf_b, std::integral_constant<int, NBLK>{}));
        }
    } else {
        // 4-byte chunks: one code group (WPG words) at a time
        for (; g < n_groups; g += n_waves) {
            float acc = 0.f;
            const int ncg = nch / WPG;
            for (int cg = 0; cg < ncg; ++cg) {
                uint32_t w[WPG];
#pragma unroll
                for (int u = 0; u < WPG; ++u)
                    w[u] = reinterpret_cast<const uint32_t*>(codes_l)[((size_t)g * nch + cg * WPG + u) * 64 + lane];
                acc = add_group<LUT, BITS>(acc, lut, w, cg * SPG, fp8);
                if (prune && ((cg + 1) * SPG) % 16 == 0 && cg + 1 < ncg && ballot64(__float_as_uint(acc) <= bound) == 0) break;
            }
            store_R(g, acc);
        }
    }
    if (filtered) flush_stage();
    else if (bounded) bound_of_nearest(a, q, len, smem, least, largest);
}

// Steps 2-3 only: the table of one pair, copied out of LDS byte for byte.
template <int LUT>
__global__ void __launch_bounds__(256)
dump_lut_kernel(const float* __restrict__ query, const float* __restrict__ centroid,
                const float* __restrict__ codebooks, int d, int pq_dim, int m, int bits, Fp8Mode fp8,
                unsigned char* __restrict__ out) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int n_entries = pq_dim << bits;
    const size_t lut_bytes = (size_t)n_entries * LutTraits<LUT>::bytes;
    unsigned char* lut = smem;
    float* rq = reinterpret_cast<float*>(smem + ((lut_bytes + 15) & ~(size_t)15));
    uint32_t* max_slot = reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(rq) + (((size_t)d * 4 + 15) & ~(size_t)15));
    for (int t = threadIdx.x; t < d; t += blockDim.x) rq[t] = query[t] - centroid[t];
    __syncthreads();
    switch (bits) {
        case 8: (void)stage_table<LUT, 8>(codebooks, rq, pq_dim, m, lut, max_slot, fp8, 0, pq_dim); break;
        case 7: (void)stage_table<LUT, 7>(codebooks, rq, pq_dim, m, lut, max_slot, fp8, 0, pq_dim); break;
        case 6: (void)stage_table<LUT, 6>(codebooks, rq, pq_dim, m, lut, max_slot, fp8, 0, pq_dim); break;
        case 5: (void)stage_table<LUT, 5>(codebooks, rq, pq_dim, m, lut, max_slot, fp8, 0, pq_dim); break;
        default: (void)stage_table<LUT, 4>(codebooks, rq, pq_dim, m, lut, max_slot, fp8, 0, pq_dim); break;
    }
    for (size_t i = threadIdx.x; i < lut_bytes / 4; i += blockDim.x)
        reinterpret_cast<uint32_t*>(out)[i] = reinterpret_cast<const uint32_t*>(lut)[i];
}

// ================================================================================================
// The (query, probe) pairs of the filtered scan grouped by cluster (a counting sort: count, offsets,
// scatter; the order inside a cluster is whatever the atomics give and does not affect any result).
// ================================================================================================
// Plain streaming read: every thread loads 16-byte words grid-strided and folds them into one word
// per workgroup.  It measures the read rate this chip's HBM reaches for the simplest possible access
// pattern - the ceiling a code scan that streams every byte from HBM could attain.
__global__ void __launch_bounds__(256) stream_read_kernel(const uint4* __restrict__ p, size_t n16, uint32_t* __restrict__ out) {
    uint4 acc = make_uint4(0u, 0u, 0u, 0u);
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) {
        const uint4 v = p[i];
        acc.x ^= v.x; acc.y ^= v.y; acc.z ^= v.z; acc.w ^= v.w;
    }
    uint32_t x = acc.x ^ acc.y ^ acc.z ^ acc.w;
    for (int o = 32; o > 0; o >>= 1) x ^= __shfl_xor(x, o);
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = part[0] ^ part[1] ^ part[2] ^ part[3];
}

// Pairs whose cluster cannot hold a vector with R <= bound.  Every decoded residual y of the cluster has |y| <= its radius,
// so |r - y| >= |r| - radius, and a vector with R <= bound has |r - y|^2 <= bound * scale + add (filter_bound) unless an
// entry of its sum saturated, which alone makes R >= top.  The counting pass marks such a pair (its distance turned negative); the
// scatter leaves it out.  (10^7 vectors, 50 probes, k = 100, 2,000 Gaussian components: 74 % of the pairs.)
struct PairCull {
    float* probe_dists;             // null: no pair is left out
    const uint32_t* bounds;
    const float* radii2;            // [n_lists] largest |y|^2
    float scale, add, top;
    __device__ bool keep(uint32_t i, int n_probes, uint32_t l) const {
        if (!probe_dists) return true;
        const uint32_t q = i / (uint32_t)(n_probes - 1), p = 1 + i - q * (uint32_t)(n_probes - 1);
        float* const at = probe_dists + (size_t)q * n_probes + p;
        const uint32_t bnd = bounds[q];
        const float rr = *at, bound = __uint_as_float(bnd);
        const float gap = __builtin_sqrtf(rr) * kCullNear - __builtin_sqrtf(radii2[l]) * kCullRadius;
        const bool out = bnd < 0x7F800000u && bound < top * kCullTop && gap > 0.f && gap * gap > __builtin_fmaf(bound, scale, add) * kCullLimit && rr < 1.0e30f;
        if (out) *at = -1.f;
        return !out;
    }
    __device__ bool kept(uint32_t i, int n_probes) const {
        if (!probe_dists) return true;
        const uint32_t q = i / (uint32_t)(n_probes - 1), p = 1 + i - q * (uint32_t)(n_probes - 1);
        return !(probe_dists[(size_t)q * n_probes + p] < 0.f);
    }
};

__global__ void pair_count_kernel(const uint4* __restrict__ pairs, uint32_t n_pairs, int n_probes, int n_lists,
                                  uint32_t* __restrict__ counts, PairCull cull) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_pairs) return;
    const uint32_t q = i / (uint32_t)(n_probes - 1), p = 1 + i - q * (uint32_t)(n_probes - 1);
    const uint32_t l = pairs[(size_t)q * n_probes + p].x;
    const uint32_t at = l < (uint32_t)n_lists ? l : 0u;           // a caller-given probe may be out of range
    if (cull.keep(i, n_probes, at)) atomicAdd(&counts[at], 1u);
}

// The same two steps for few clusters, where many pairs name the same cluster and one global atomic per
// pair would serialise: a workgroup of 1024 threads takes `chunk` pairs, counts them per cluster in LDS
// and issues one global atomic per cluster it met.  Dynamic LDS: n_lists words (count) or 2 n_lists (scatter).
// Pairs a workgroup takes: a workgroup walks through its share 1,024 at a time, each step waiting for the one before, so the share is what
// leaves one for every compute unit.  Both kernels, us, at 24 / 64 / 128 / 256 workgroups aimed at: 190,000 pairs of 1,024 clusters
// 26 / 15 / 14 / 15, 237,000 of 5,000 29 / 24 / 20 / 18, 630,000 of 2,000 37 / 36 / 29 / 28, 261,000 of 8,000 31 / 21 / 17 / 14; 25,000 of 1,024
// 24 at four workgroups, 10 at 25.
inline uint32_t pair_chunk(size_t n_pairs) {
    const size_t share = (n_pairs / 256 + 1023) / 1024 * 1024;
    return (uint32_t)std::min<size_t>(std::max<size_t>(share, 1024), 8192);
}
constexpr int kPairLdsLists = 8192;       // up to this many clusters

__device__ inline uint32_t pair_cluster(const uint4* __restrict__ pairs, uint32_t i, int n_probes, int n_lists) {
    const uint32_t q = i / (uint32_t)(n_probes - 1), p = 1 + i - q * (uint32_t)(n_probes - 1);
    const uint32_t l = pairs[(size_t)q * n_probes + p].x;
    return l < (uint32_t)n_lists ? l : 0u;                        // a caller-given probe may be out of range
}

// What the grouped order holds of pair i: its number, or (records given) what the matrix-core filter works from, {query, slot
// of the probe, squared distance to the centroid, bound}, so that a work item's pairs are one read.
struct PairRecords {
    uint4* records;
    const float* probe_dists;
    const uint32_t* bounds;
};
__device__ inline void store_pair(uint32_t at, uint32_t i, int n_probes, uint32_t* __restrict__ order, const PairRecords& r) {
    if (!r.records) { order[at] = i; return; }
    const uint32_t q = i / (uint32_t)(n_probes - 1), p = 1 + i - q * (uint32_t)(n_probes - 1);
    r.records[at] = make_uint4(q, p, __float_as_uint(r.probe_dists[(size_t)q * n_probes + p]), r.bounds[q]);
}

__global__ void __launch_bounds__(1024)
pair_count_lds_kernel(const uint4* __restrict__ pairs, uint32_t n_pairs, uint32_t chunk, int n_probes, int n_lists,
                      uint32_t* __restrict__ counts, PairCull cull) {
    extern __shared__ uint32_t s_cnt[];
    for (int l = threadIdx.x; l < n_lists; l += blockDim.x) s_cnt[l] = 0;
    __syncthreads();
    const uint32_t i0 = blockIdx.x * chunk, i1 = i0 + chunk < n_pairs ? i0 + chunk : n_pairs;
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
        const uint32_t l = pair_cluster(pairs, i, n_probes, n_lists);
        if (cull.keep(i, n_probes, l)) atomicAdd(&s_cnt[l], 1u);
    }
    __syncthreads();
    for (int l = threadIdx.x; l < n_lists; l += blockDim.x)
        if (s_cnt[l]) atomicAdd(&counts[l], s_cnt[l]);
}

__global__ void __launch_bounds__(1024)
pair_scatter_lds_kernel(const uint4* __restrict__ pairs, uint32_t n_pairs, uint32_t chunk, int n_probes, int n_lists,
                        const uint32_t* __restrict__ offsets, uint32_t* __restrict__ cursor, uint32_t* __restrict__ order, PairRecords rec, PairCull cull) {
    extern __shared__ uint32_t s_mem[];
    uint32_t* s_cnt = s_mem;                  // pairs of this chunk per cluster, then the running rank
    uint32_t* s_base = s_mem + n_lists;       // first slot of this chunk's pairs inside the cluster's range
    for (int l = threadIdx.x; l < n_lists; l += blockDim.x) s_cnt[l] = 0;
    __syncthreads();
    const uint32_t i0 = blockIdx.x * chunk, i1 = i0 + chunk < n_pairs ? i0 + chunk : n_pairs;
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += blockDim.x)
        if (cull.kept(i, n_probes)) atomicAdd(&s_cnt[pair_cluster(pairs, i, n_probes, n_lists)], 1u);
    __syncthreads();
    for (int l = threadIdx.x; l < n_lists; l += blockDim.x) {
        const uint32_t c = s_cnt[l];
        s_base[l] = c ? offsets[l] + atomicAdd(&cursor[l], c) : 0u;
        s_cnt[l] = 0;
    }
    __syncthreads();
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
        if (!cull.kept(i, n_probes)) continue;
        const uint32_t l = pair_cluster(pairs, i, n_probes, n_lists);
        store_pair(s_base[l] + atomicAdd(&s_cnt[l], 1u), i, n_probes, order, rec);
    }
}

// offsets[l] = counts[0] + ... + counts[l-1]; one workgroup, 4096 counters per trip: four consecutive
// counters per thread (coalesced), a scan inside each wave, the 16 wave totals through LDS
__global__ void __launch_bounds__(1024)
pair_offsets_kernel(const uint32_t* __restrict__ counts, int n_lists, uint32_t* __restrict__ offsets) {
    __shared__ uint32_t wave_total[16];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    uint32_t carry = 0;
    for (int base = 0; base < n_lists; base += 4096) {
        const int i = base + tid * 4;
        uint32_t c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = i + u < n_lists ? counts[i + u] : 0u;
        const uint32_t own = c[0] + c[1] + c[2] + c[3];
        const uint32_t incl = wave_inclusive_scan(own);
        if (lane == kWave - 1) wave_total[wave] = incl;
        __syncthreads();
        uint32_t before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const uint32_t t = wave_total[w];
            before += w < wave ? t : 0u;
            total += t;
        }
        uint32_t at = carry + before + incl - own;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (i + u < n_lists) offsets[i + u] = at;
            at += c[u];
        }
        carry += total;
        __syncthreads();
    }
}

__global__ void pair_scatter_kernel(const uint4* __restrict__ pairs, uint32_t n_pairs, int n_probes, int n_lists,
                                    const uint32_t* __restrict__ offsets, uint32_t* __restrict__ cursor,
                                    uint32_t* __restrict__ order, PairRecords rec, PairCull cull) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_pairs || !cull.kept(i, n_probes)) return;
    const uint32_t q = i / (uint32_t)(n_probes - 1), p = 1 + i - q * (uint32_t)(n_probes - 1);
    uint32_t l = pairs[(size_t)q * n_probes + p].x;
    if (l >= (uint32_t)n_lists) l = 0u;
    store_pair(offsets[l] + atomicAdd(&cursor[l], 1u), i, n_probes, order, rec);
}

// Work items of the matrix-core filter, and the place of every cluster's pairs in the grouped order (any disjoint ranges
// will do): 64 clusters per workgroup, their ranges taken with one addition each; its 16 waves write the items, one cluster after the
// other.  per_item: vectors of an item.  totals: pairs, items.
__global__ void __launch_bounds__(1024)
filter_items_kernel(const uint32_t* __restrict__ counts, const uint32_t* __restrict__ list_sizes, const int64_t* __restrict__ group_offsets,
                    int n_lists, uint32_t per_item, uint32_t* __restrict__ offsets, uint32_t* __restrict__ totals, uint4* __restrict__ items, uint32_t cap) {
    __shared__ uint32_t s_base[2];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), l = blockIdx.x * kWave + lane;
    const uint32_t n = l < n_lists ? counts[l] : 0u, len = l < n_lists ? list_sizes[l] : 0u, group = l < n_lists ? (uint32_t)group_offsets[l] : 0u;
    const uint32_t tiles = (n + (uint32_t)kFilterPairs - 1u) / (uint32_t)kFilterPairs, chunks = (len + per_item - 1u) / per_item;
    const uint32_t mine = tiles * chunks, upto_n = wave_inclusive_scan(n), upto_items = wave_inclusive_scan(mine);
    if (threadIdx.x == kWave - 1) {
        s_base[0] = upto_n ? atomicAdd(&totals[0], upto_n) : 0u;
        s_base[1] = upto_items ? atomicAdd(&totals[1], upto_items) : 0u;
    }
    __syncthreads();
    const uint32_t first = s_base[0] + upto_n - n, at = s_base[1] + upto_items - mine;
    if (wave == 0 && n != 0) offsets[l] = first;
    for (int s = wave; s < kWave; s += 16) {
        auto of = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, s); };
        const uint32_t mine_s = of(mine);
        if (mine_s == 0) continue;
        const uint32_t n_s = of(n), first_s = of(first), tiles_s = of(tiles), at_s = of(at), l_s = of((uint32_t)l), len_s = of(len), group_s = of(group);
        for (uint32_t i = (uint32_t)lane; i < mine_s; i += kWave) {
            const uint32_t c = i / tiles_s, t = i - c * tiles_s;       // the items that read the same codes are neighbours
            const uint32_t done = t * (uint32_t)kFilterPairs, n_here = n_s - done < (uint32_t)kFilterPairs ? n_s - done : (uint32_t)kFilterPairs;
            const uint32_t v0 = c * per_item, v_here = len_s - v0 < per_item ? len_s - v0 : per_item;
            if (at_s + i < cap) {
                items[2 * (size_t)(at_s + i)] = make_uint4(l_s, first_s + done, n_here, v_here);
                items[2 * (size_t)(at_s + i) + 1] = make_uint4(v0, group_s + v0 / 64u, 0u, 0u);
            }
        }
    }
}

// The queries in the order of their nearest clusters, in one launch: a workgroup goes over the nearest cluster of every query (left by the
// selection), ranks those of its own 64 clusters, counts those of the clusters before, and writes its queries.  5 us for 10,000
// queries and 1,024 or 10,000 clusters; one workgroup for all of them took over 100.
using ivfpq::kNearestPerThread;
__global__ void __launch_bounds__(1024)
nearest_order_kernel(const uint32_t* __restrict__ nearest, int nq, uint32_t* __restrict__ order) {
    __shared__ uint32_t s_count[kWave], s_before;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t l0 = blockIdx.x * kWave;
    uint32_t mine[kNearestPerThread];                                // cluster less l0
#pragma unroll
    for (int u = 0; u < kNearestPerThread; ++u) {
        const int q = u * 1024 + tid;
        mine[u] = q < nq ? nearest[q] : 0xFFFFFFFFu;
    }
    if (tid < kWave) s_count[tid] = 0u;
    if (tid == 0) s_before = 0u;
    __syncthreads();
    uint32_t before = 0, rank[kNearestPerThread];
#pragma unroll
    for (int u = 0; u < kNearestPerThread; ++u) {
        before += mine[u] < l0 ? 1u : 0u;
        mine[u] -= l0;                                               // (of no query: far above 64 still)
        rank[u] = mine[u] < (uint32_t)kWave ? atomicAdd(&s_count[mine[u]], 1u) : 0u;
    }
    before = wave_inclusive_scan(before);
    if (lane == kWave - 1 && before != 0) atomicAdd(&s_before, before);
    __syncthreads();
    const uint32_t n = s_count[lane], first = s_before + wave_inclusive_scan(n) - n;
    __syncthreads();
    if (wave == 0) s_count[lane] = first;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kNearestPerThread; ++u)
        if (mine[u] < (uint32_t)kWave) order[s_count[mine[u]] + rank[u]] = (uint32_t)(u * 1024 + tid);
}

// ================================================================================================
// Step 5: the k smallest (R, id) of a query.  Candidates: the survivor list of the filtered scan (listed: the nearest
// cluster's values under the bound, then what the scan kept), or the segments of all probes themselves.
// ================================================================================================
template <int CAP, int THREADS>          // record capacity, >= k
__global__ void __launch_bounds__(THREADS)
topk_kernel(const float* __restrict__ R, const uint32_t* __restrict__ Rpos, size_t stride,
            const uint32_t* __restrict__ roff, const uint32_t* __restrict__ probes,
            const uint32_t* __restrict__ bounds, const uint32_t* __restrict__ counts, int n_probes, int n_lists, int k,
            const int64_t* __restrict__ list_offsets, const int64_t* __restrict__ ids,
            int64_t* __restrict__ out_ids, float* __restrict__ out_dists, bool listed) {
    __shared__ RowSelectSharedT<CAP> t;
    // where the segments of up to kInLds probes start and their clusters' first ids: a survivor's search and id are then one read from
    // global memory instead of a chain of nine
    constexpr int kInLds = 128;
    __shared__ uint32_t l_roff[kInLds];
    __shared__ long long l_first[kInLds];
    auto& s = t.sel;
    const int q = blockIdx.x;
    const int tid = threadIdx.x, nth = blockDim.x;
    const uint32_t* s_roff = roff + (size_t)q * (n_probes + 1);
    const uint32_t* s_probe = probes + (size_t)q * n_probes;
    const bool in_lds = n_probes <= kInLds;
    if (in_lds)
        for (int p = tid; p < n_probes; p += nth) {
            const uint32_t l = s_probe[p];
            l_roff[p] = s_roff[p];
            l_first[p] = l < (uint32_t)n_lists ? (long long)list_offsets[l] : 0ll;         // (a caller-given probe out of range has no vectors)
        }
    const uint32_t seg0 = s_roff[1];          // padded length of the nearest probe's segment (a multiple of 64)
    const uint32_t n = listed ? counts[q] : s_roff[n_probes];
    const uint32_t* row = reinterpret_cast<const uint32_t*>(R + (size_t)q * stride) + (listed ? seg0 : 0u);
    const uint32_t* row_pos = Rpos + (size_t)q * stride + (listed ? seg0 : 0u);

    // position of candidate i in the unfiltered layout (probe segments back to back)
    auto pos_of = [&](uint32_t i) { return listed ? row_pos[i] : i; };
    // tie key = the caller's id of the candidate at that position (padding slots sort last)
    auto id_of = [&](uint32_t pos, uint32_t key) -> long long {
        if (key == kPadKey) return 0x7FFFFFFFFFFFFFFFll;
        int lo = 0, hi = n_probes;            // largest probe slot with roff[slot] <= pos
        if (in_lds) {
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (l_roff[mid] <= pos) lo = mid; else hi = mid;
            }
            return (long long)ids[l_first[lo] + (long long)(pos - l_roff[lo])];
        }
        while (hi - lo > 1) {
            int mid = (lo + hi) >> 1;
            if (s_roff[mid] <= pos) lo = mid; else hi = mid;
        }
        return (long long)ids[list_offsets[s_probe[lo]] + (int64_t)(pos - s_roff[lo])];
    };
    // The survivor list was filtered by the query's bound already, so that bound weeds out nothing here: the
    // selection takes its own from a sample of the list (the k-th smallest of its first entries), and one pass over
    // the list with that bound leaves a few hundred candidates.
    const int got = block_select_row(t, row, n, (uint32_t)k, false, 0u, pos_of, id_of);
    for (int j = tid; j < k; j += nth) {
        int64_t id = -1;
        float dist = __uint_as_float(0x7F800000u);
        if (j < got && s.rec_key[j] != kPadKey) { id = (int64_t)s.rec_tie[j]; dist = __uint_as_float(s.rec_key[j]); }
        out_ids[(size_t)q * k + j] = id;
        out_dists[(size_t)q * k + j] = dist;
    }
}

// ================================================================================================
// Re-ranking with the stored vectors: per query the exact squared distances of its candidates (fp32,
// direct form) and the k smallest by (distance, id).  One workgroup per query; a group of 8 adjacent
// lanes per candidate (each lane sums every 8th component, then three exchange steps: a fixed order).
// Candidate ids outside [0, n_data) are skipped.
// ================================================================================================
__global__ void __launch_bounds__(SEL_THREADS)
refine_kernel(const float* __restrict__ data, long long n_data, int d, const float* __restrict__ queries,
              const int64_t* __restrict__ cand, int n_cand, int k, int64_t* __restrict__ out_ids,
              float* __restrict__ out_dists) {
    __shared__ SelectShared s;
    __shared__ uint32_t keys[SEL_CAP];
    const int q = blockIdx.x;
    const int tid = threadIdx.x, nth = blockDim.x;
    const float* qv = queries + (size_t)q * d;
    const int64_t* my = cand + (size_t)q * n_cand;
    for (int base = 0; base < n_cand; base += nth / 8) {
        const int c = base + (tid >> 3);
        const bool valid = c < n_cand;
        const long long id = valid ? (long long)my[c] : -1ll;
        const bool ok = id >= 0 && id < n_data;
        float acc = 0.f;
        if (ok) {
            const float* x = data + (size_t)id * d;
            for (int u = tid & 7; u < d; u += 8) { const float diff = qv[u] - x[u]; acc = __builtin_fmaf(diff, diff, acc); }
        }
        acc = sum_over_8_lanes(acc);
        if (valid && (tid & 7) == 0) keys[c] = ok ? __float_as_uint(acc) : kPadKey;
    }
    __syncthreads();
    const int got = block_select_smallest(s, (uint32_t)n_cand, (uint32_t)k,
        [&](uint32_t i) { return keys[i]; },
        [&](uint32_t i) { return keys[i] == kPadKey ? 0x7FFFFFFFFFFFFFFFll : (long long)my[i]; });
    for (int j = tid; j < k; j += nth) {
        int64_t id = -1;
        float dist = __uint_as_float(0x7F800000u);
        if (j < got && s.rec_key[j] != kPadKey) { id = (int64_t)s.rec_tie[j]; dist = __uint_as_float(s.rec_key[j]); }
        out_ids[(size_t)q * k + j] = id;
        out_dists[(size_t)q * k + j] = dist;
    }
}

// ================================================================================================
// Host side
// ================================================================================================
struct ImageLayout {
    size_t centroids, centroid_norms, codebooks, word_norms, list_offsets, list_sizes, list_radii, group_offsets, codes, ids, total;
};

int chunk_width(const ivfpq_index* idx) {
    const int cb = idx->code_bytes(), p = idx->pq_bits;
    const bool wide = cb % 16 == 0 && cb / 16 <= 4 && (p == 4 || p == 8 || (p == 6 && cb == 48));
    return wide ? 16 : 4;
}

ImageLayout image_layout(const ivfpq_index* idx) {
    ImageLayout L{};
    size_t at = 0;
    auto take = [&](size_t bytes) { size_t o = at; at = align_up(at + bytes); return o; };
    L.centroids = take(idx->centroids.size() * sizeof(float));
    L.centroid_norms = take((size_t)idx->n_lists * sizeof(float));
    L.codebooks = take(idx->codebooks.size() * sizeof(float));
    L.word_norms = take(((size_t)idx->pq_dim << idx->pq_bits) * sizeof(float));
    L.list_offsets = take(((size_t)idx->n_lists + 1) * sizeof(int64_t));
    L.list_sizes = take((size_t)idx->n_lists * sizeof(uint32_t));
    L.list_radii = take((size_t)idx->n_lists * sizeof(float));
    L.group_offsets = take(((size_t)idx->n_lists + 1) * sizeof(int64_t));
    L.codes = take((size_t)idx->total_groups * 64 * idx->code_bytes());
    // (the ids' place holds the codes in transit during the upload: one group at least)
    L.ids = take(idx->n == 0 ? 0 : std::max((size_t)idx->n * sizeof(int64_t), (size_t)64 * idx->code_bytes()));
    L.total = at == 0 ? kAlign : at;
    return L;
}

struct Plan {
    int64_t tile;           // queries per tile
    size_t stride;          // R slots per query
    size_t probes, probe_d, roff, pairs, bounds, counts, D, S, split, R, Rpos, order, list_counts, list_cursor, list_offsets, total;
};


// Vectors of a work item: as many as leave every wave of the chip (eight per compute unit) two items to take, lists of average length
// reckoned (32 lists of 1,900 vectors, 3,500 pairs: 256 items of 512 vectors took 93 us).
uint32_t filter_item_vectors(const ivfpq_index* idx, size_t n_pairs) {
    const double tiles = (double)n_pairs / kFilterPairs + 0.5 * (double)std::min<size_t>(n_pairs, (size_t)idx->n_lists);
    uint32_t v = kFilterVectors;
    while (v > 64 && tiles * ((double)idx->n / (double)idx->n_lists / v + 0.5) < 4096.0) v /= 2;
    return v;
}
// How many can be needed: a cluster of c pairs and v vectors has ceil(c / 64) ceil(v / per_item).
size_t filter_items_max(const ivfpq_index* idx, size_t n_pairs, uint32_t per_item) {
    const size_t longest = idx->sorted_padded_sizes.empty() ? 0 : idx->sorted_padded_sizes[0];
    const size_t chunks = (longest + per_item - 1) / per_item;
    return n_pairs / kFilterPairs * chunks + chunks + (size_t)idx->total_groups * 64 / per_item + (size_t)idx->n_lists;
}
// The filter's lists in the workspace: a query's starting length, totals, pairs, work items (offsets from the place of the ranking values).
struct FilterLists {
    uint32_t per_item;
    size_t max_items, totals, records, items, bytes;
};
FilterLists filter_lists(const ivfpq_index* idx, size_t nq, int n_probes, uint32_t per_item) {
    FilterLists f;
    const size_t n_pairs = nq * (size_t)(n_probes - 1);
    f.per_item = per_item;
    f.max_items = filter_items_max(idx, n_pairs, f.per_item);
    f.totals = align_up(nq * 4);
    f.records = f.totals + kAlign;
    f.items = f.records + align_up(n_pairs * sizeof(uint4));
    f.bytes = f.items + align_up(f.max_items * 2 * sizeof(uint4));
    return f;
}

// Vectors looked up beyond the nearest probes' from which the matrix-core filter pays at the earliest (filter_pays).
constexpr double kFilterLookups = 5e6;

// Places of a tile's arrays.  need_D: clusters are ranked (the caller gives none); with_filter: the filter's lists have room.
void lay_out(const ivfpq_index* idx, int64_t tile, int32_t n_probes, bool need_D, bool with_filter, Plan* plan) {
    const size_t strips = ((size_t)idx->n_lists + 31) / 32;      // strip summaries of the ranking keys, narrowest strips
    plan->tile = tile;
    size_t at = 0;
    auto take = [&](size_t bytes) { size_t o = at; at = align_up(at + bytes); return o; };
    plan->probes = take((size_t)tile * n_probes * 4);
    plan->probe_d = take((size_t)tile * n_probes * 4);
    plan->roff = take((size_t)tile * (n_probes + 1) * 4);
    plan->pairs = take((size_t)tile * n_probes * 16);
    plan->bounds = take((size_t)tile * 4);
    plan->counts = take((size_t)tile * 4);
    plan->D = take(need_D ? (size_t)tile * idx->n_lists * 4 : 0);
    plan->S = take(need_D ? (size_t)tile * strips * sizeof(StripSummary) : 0);
    plan->split = take(need_D ? coarse_split_bytes((size_t)tile, (size_t)idx->n_lists, idx->d) : 0);
    if (with_filter) {                // the filter's lists, where the ranking values leave too little room for them
        // (for items of the most vectors, so that a smaller batch never needs more than a larger one)
        const size_t want = filter_lists(idx, (size_t)tile, n_probes, kFilterVectors).bytes;
        if (want > at - plan->D) take(want - (at - plan->D));
    }
    plan->R = take((size_t)tile * plan->stride * 4);
    plan->Rpos = take((size_t)tile * plan->stride * 4);
    plan->order = take((size_t)tile * (n_probes > 1 ? n_probes - 1 : 0) * 4);
    plan->list_counts = take((size_t)idx->n_lists * 4);
    plan->list_cursor = take((size_t)idx->n_lists * 4);
    plan->list_offsets = take((size_t)idx->n_lists * 4);
    plan->total = at;
}

// given_probes: the caller chooses the clusters and may name one several times, so the bound on a
// query's candidates is n_probes times the largest cluster rather than the n_probes largest ones
// limit: the bytes the plan should stay within (0: the index's workspace limit).  The tile is the largest whose plan
// does; where one query's exceeds the limit it is one query, and the caller compares plan->total with what it has.
// A smaller batch never needs more than a larger one: what the tile holds at most, and whether the filter's lists have
// room, follow from the index, the probes and the limit alone.
int make_plan(const ivfpq_index* idx, int64_t nq, int32_t n_probes, bool given_probes, Plan* plan, size_t limit = 0) {
    if (limit == 0) limit = idx->workspace_limit;
    const bool need_D = !given_probes;
    int64_t stride = given_probes
        ? (int64_t)n_probes * (idx->sorted_padded_sizes.empty() ? 0 : idx->sorted_padded_sizes[0])
        : idx->max_padded_candidates(n_probes);
    // the survivor list of a query also takes the nearest cluster's values under the bound
    stride += idx->sorted_padded_sizes.empty() ? 0 : idx->sorted_padded_sizes[0];
    if (stride >= ((int64_t)1 << 31))
        return fail(IVFPQ_EUNSUPPORTED, "a query may see %lld candidates (limit 2^31)", (long long)stride);
    plan->stride = (size_t)std::max<int64_t>(stride, 64);
    // An estimate of the tile: what a query takes, and what does not grow with the tile (three per-cluster counter arrays, the
    // centroids' bf16 halves, alignment slack).  128: the query rows' padding.
    const size_t strips = ((size_t)idx->n_lists + 31) / 32;
    const size_t per_query = plan->stride * 8 + (need_D ? ((size_t)idx->n_lists + 4 * strips + coarse_padded_dim(idx->d)) * 4 : 0) +
                             (size_t)n_probes * 28 + 16;      // probe lists, distances, offsets, descriptors, order, bound, counter
    const size_t fixed = 3 * align_up((size_t)idx->n_lists * 4)
                         + (need_D ? coarse_split_bytes(128, (size_t)idx->n_lists, idx->d) : 0) + 24 * kAlign;
    const int64_t most = std::max<int64_t>(1, limit > fixed ? (int64_t)((limit - fixed) / per_query) : 1);
    // The filter's lists: where it is built for the index and a tile can hold enough work for it.
    bool with_filter = need_D && n_probes > 1 && filter_supported(idx->pq_bits, idx->pq_dim, idx->d, chunk_width(idx)) &&
                       (double)most * (n_probes - 1) * (double)idx->n / (double)idx->n_lists >= kFilterLookups;
    auto fits = [&](int64_t tile) {
        lay_out(idx, tile, n_probes, need_D, with_filter, plan);
        return plan->total <= limit;
    };
    int64_t tile = std::min(most, std::max<int64_t>(nq, 1));
    if (fits(tile)) return IVFPQ_OK;
    if (with_filter && !fits(1)) {          // one query that fits the limit only without them does without
        with_filter = false;
        if (fits(tile)) return IVFPQ_OK;
    }
    // the estimate leaves out what the filter's work items and paddings take: a few per cent
    int64_t lo = 1, hi = tile;              // the largest tile that fits is in [lo, hi), or is one query
    while (hi - lo > 1) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (fits(mid)) lo = mid; else hi = mid;
    }
    (void)fits(lo);
    return IVFPQ_OK;
}

int check_search_args(const ivfpq_index* idx, const void* q, int64_t nq, int32_t n_probes, int32_t k,
                      int32_t lut_dtype, bool need_k) {
    if (!idx) return fail(IVFPQ_EINVAL, "null index");
    if (nq < 0) return fail(IVFPQ_EINVAL, "nq=%lld", (long long)nq);
    if (nq > 0 && !q) return fail(IVFPQ_EINVAL, "null queries");
    if (n_probes < 1 || n_probes > idx->n_lists || n_probes > IVFPQ_MAX_PROBES)
        return fail(IVFPQ_EINVAL, "n_probes=%d outside [1, min(n_lists=%d, %d)]", n_probes, idx->n_lists, IVFPQ_MAX_PROBES);
    if (need_k && (k < 1 || k > IVFPQ_MAX_K)) return fail(IVFPQ_EINVAL, "k=%d outside [1, %d]", k, IVFPQ_MAX_K);
    if (lut_dtype < 0 || lut_dtype > 3) return fail(IVFPQ_EINVAL, "unknown lut_dtype %d", lut_dtype);
    return IVFPQ_OK;
}

size_t lut_elem_bytes(int lut_dtype) { return lut_dtype == IVFPQ_LUT_FP32 ? 4 : (lut_dtype == IVFPQ_LUT_FP16 ? 2 : 1); }

size_t scan_lds_bytes(const ivfpq_index* idx, int lut_dtype) {
    size_t lut = (size_t)idx->pq_dim * idx->ksub() * lut_elem_bytes(lut_dtype);
    return ((lut + 15) & ~(size_t)15) + (((size_t)idx->d * 4 + 15) & ~(size_t)15) + 16;
}
// plus the per-wave survivor staging of the filtered scan
size_t scan_lds_bytes_staged(const ivfpq_index* idx, int lut_dtype, int threads) {
    return scan_lds_bytes(idx, lut_dtype) + (size_t)(threads / 64) * (kStageCap * 8 + kAliveCap * 2)
           + (size_t)idx->tuning.lds_pad;      // the pad sits behind everything the kernel addresses
}

int check_device(const ivfpq_index* idx) {
    if (!idx->dev.valid) return fail(IVFPQ_ESTATE, "index has no device image: call ivfpq_upload first");
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != idx->dev.device)
        return fail(IVFPQ_ESTATE, "index was uploaded to device %d, current device is %d", idx->dev.device, dev);
    return IVFPQ_OK;
}

int scan_threads(const ivfpq_index* idx, int lut_dtype) {
    if (idx->tuning.scan_threads) return idx->tuning.scan_threads;       // validated by ivfpq_set_tuning
    // measured on MI355X: small tables want many 4-wave workgroups per CU; large tables want the
    // largest workgroup of which two still fit the CU's LDS (table + residual + survivor staging);
    // long lists (24 or more 64-vector groups on average) want 2-wave workgroups: the table build of
    // one pair then overlaps the scan of more others
    size_t lds = scan_lds_bytes(idx, lut_dtype);
    if (idx->n_lists > 0 && idx->n / idx->n_lists >= 24 * 64 && lds <= 24 * 1024) return 128;
    if (lds <= 32 * 1024) return 256;       // (half table, 48 sub-spaces, 29 KB: 1.19 ms with 256 threads, 1.26 with 512)
    if (lds <= 40 * 1024) return 512;
    if (2 * (lds + (size_t)16 * kStageCap * 8) <= kLdsBytes) return 1024;
    return 512;
}

constexpr size_t kWaveSlots = 256 * 32;  // waves the chip holds at once
constexpr uint32_t kOrderBlock = 64;     // consecutive pairs of the grouped order that stay on one XCD

// How the probes of a tile are scanned, by the number of vectors that are looked up (lists of average length):
//   kWholeRows  every value of every probe is written and the top-k step reads them all: one scan launch in place of
//               the nearest probe's, the bound's, the grouping's and the others'.  Up to 16,384 vectors a query and
//               3.2 M in all.
//   kInOrder    the filtered scan takes its pairs query by query: up to 6 M vectors the grouping costs more than
//               shared clusters and tables give back.
//   kGrouped    pairs grouped by cluster, which pays in batches (scan stage of 10,000 queries at 10^8 vectors 10.4 ->
//               6.8 ms, at 10^7 1.91 -> 1.51; and always beyond 2^20 pairs, of lists that are nearly empty).
// Measured, us a search (M: vectors looked up by this reckoning; whole rows / in order / grouped with the table kernels, when the
// grouping took 14 us more than it does; now the two are even at 6 M: 75 / 76, 75 / 75, 94 / 84, 72 / 68, 95 / 82, in order / grouped):
//   64 sub-spaces of 8 bits, e5m3, lists of 1,000    5 probes: 2.5 M 106 / 108 / 113, 5 M 163 / 138 / 144
//                                                    20 probes: 5 M 156 / 115 / 126, 10 M 265 / 164 / 170, 20 M - / 264 / 251
//   48 of 8 bits, half                               5 probes: 2.5 M 71 / 80 / 87, 5 M 113 / 111 / 117; 20: 10 M 171 / 142 / 140
//   64 of 4 bits, half, lists of 2,000               5 probes: 2.6 M 127 / 153 / 218, 5.1 M 195 / 198 / 239, 10 M 408 / 306 / 296
//   64 of 7 bits, e5m3                               5 probes: 2.5 M 101 / 104 / 126, 5 M 156 / 140 / 146; 20: 10 M 251 / 181 / 167
//   32 of 8 bits, float                              5 probes: 5 M 144 / 143 / 145, 10 M 243 / 219 / 214; 33: 8 M 182 / 168 / 161
//   more than 16,384 a query, one query              33 probes, float 46 / 38 / 52; 20 of 2,000, 4 bits 82 / 45 / 176
// Lists of average length on purpose, also where they are uneven: the filtered routes wait there for one workgroup per
// query that walks the longest list and then for its bound, which costs more than the values the filter saves
// (10^6 vectors, the longest list 134,000: 5 probes, 64 / 256 queries 311 / 446 us whole, 856 / 1067 in order; 5 probes of
// which one has 290,000: 472 / 876 and 2156 / 2646).  Reckoned by the length of the list that a vector lies in (sum of
// len^2 / n) these searches would leave the whole rows, and lose.
// A caller may name the route (IVFPQ_TUNE_SCAN_ROUTE); one that sets a knob of the grouped scan alone gets that.
enum class ScanRoute { kWholeRows = 1, kInOrder = 2, kGrouped = 3 };
ScanRoute scan_route(const ivfpq_index* idx, int nq, int n_probes) {
    const ivfpq::Tuning& t = idx->tuning;
    const size_t pairs = (size_t)nq * n_probes;
    if (t.scan_route != 0 && pairs <= 0x7FFFFFFFull) return (ScanRoute)t.scan_route;      // a workgroup per pair: one dimension of a grid
    if (t.order_block != 0 || t.scan_share != 0 || pairs > ((size_t)1 << 20)) return ScanRoute::kGrouped;
    const double per_query = (double)n_probes * (double)idx->n / (double)idx->n_lists, all = per_query * nq;
    if (per_query <= 16384.0 && all <= 3.2e6) return ScanRoute::kWholeRows;
    return all <= 6e6 ? ScanRoute::kInOrder : ScanRoute::kGrouped;
}

bool group_pairs_by_cluster(size_t n_pairs) { return n_pairs < ((size_t)1 << 32) - 8 * (size_t)kOrderBlock; }

template <int LUT, int BITS>
int launch_scan_bits(const ScanArgs& a, int cw, int nch, dim3 grid, int threads, size_t lds, hipStream_t st) {
    auto go = [&](auto kernel) -> int {
        if (int s = allow_full_lds(kernel)) return s;
        if (int s = require_no_static_lds(reinterpret_cast<const void*>(kernel))) return s;
        hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, st, a);
        HIP_TRY(hipGetLastError());
        return IVFPQ_OK;
    };
    if (cw == 16) {
        // 16-byte chunks need whole code groups per vector's chunk set: always true for 4- and 8-bit
        // codes; of the other widths only 6-bit codes with 48 bytes per vector qualify
        if constexpr (BITS == 4 || BITS == 8) {
            switch (nch) {
                case 1: return go(scan_kernel<LUT, BITS, 16, 1>);
                case 2: return go(scan_kernel<LUT, BITS, 16, 2>);
                case 3: return go(scan_kernel<LUT, BITS, 16, 3>);
                case 4: return go(scan_kernel<LUT, BITS, 16, 4>);
                default: break;
            }
        } else if constexpr (BITS == 6) {
            if (nch == 3) return go(scan_kernel<LUT, BITS, 16, 3>);
        }
        return fail(IVFPQ_EUNSUPPORTED, "internal: no scan kernel for %d chunks of 16 bytes of %d-bit codes", nch, BITS);
    }
    return go(scan_kernel<LUT, BITS, 4, 0>);
}

template <int LUT>
int launch_scan_lut(const ScanArgs& a, int bits, int cw, int nch, dim3 grid, int threads, size_t lds, hipStream_t st) {
    switch (bits) {
        case 8: return launch_scan_bits<LUT, 8>(a, cw, nch, grid, threads, lds, st);
        case 7: return launch_scan_bits<LUT, 7>(a, cw, nch, grid, threads, lds, st);
        case 6: return launch_scan_bits<LUT, 6>(a, cw, nch, grid, threads, lds, st);
        case 5: return launch_scan_bits<LUT, 5>(a, cw, nch, grid, threads, lds, st);
        default: return launch_scan_bits<LUT, 4>(a, cw, nch, grid, threads, lds, st);
    }
}

// ---- the group kernel: up to G pairs of one cluster per workgroup, tables interleaved entry by entry ----
size_t scan_group_lds_bytes(const ivfpq_index* idx, int lut_dtype, int G, int threads) {
    return kGroupHead + (size_t)idx->pq_dim * ((size_t)1 << idx->pq_bits) * G * lut_elem_bytes(lut_dtype) + (((size_t)G * idx->d * 4 + 15) & ~(size_t)15)
           + (size_t)(threads / 64) * (kGroupStageAll * 8 + kAliveCap * 2) + 16 + (size_t)idx->tuning.lds_pad;
}
// Workgroup size of the group kernel.  Measured on MI355X (filtered scan, 10,000 queries): with long lists (24 or
// more 64-vector groups on average) two-wave workgroups win when six or more of them share a compute unit's LDS
// (e5m3, two pairs, 10^8 vectors: 4.81 ms against 5.30 with four waves) and lose badly otherwise (half table, two
// pairs, 35 KB: 8.04 ms against 5.63).  Tables too large for four workgroups of four waves per compute unit take eight
// waves, two workgroups: the same 16 waves with half as many tables (whole search, 10,000 queries on 10^6 vectors, 256 / 512
// threads: half, 64 sub-spaces, two pairs 2.26 / 1.92 ms; float, 32 sub-spaces, two pairs 1.96 / 1.68; half, 32, four pairs
// 1.57 / 1.32; e5m3, 64, four pairs 1.89 / 1.64).
constexpr size_t kGroupLds4 = 40 * 1024, kGroupLds2 = 80 * 1024;      // LDS of a workgroup of which four / two share a compute unit
int scan_group_threads(const ivfpq_index* idx, int lut_dtype, int G) {
    if (idx->tuning.scan_threads) return std::min(idx->tuning.scan_threads, 512);       // the kernel's launch bound
    const bool long_lists = idx->n_lists > 0 && idx->n / idx->n_lists >= 24 * 64;
    if (long_lists && scan_group_lds_bytes(idx, lut_dtype, G, 128) <= 24 * 1024) return 128;
    return scan_group_lds_bytes(idx, lut_dtype, G, 256) <= kGroupLds4 ? 256 : 512;
}
// Bit-packed codes of how many sub-spaces the group kernel is built for: whole words with no more than 21 of them (two
// buffers of a vector's words beside the sums of four queries fill the registers), 16 sub-spaces aside (fewer than two
// steps).
bool scan_group_packed(int pq_bits, int pq_dim) {
    return pq_dim == 32 || pq_dim == 64 || pq_dim == 96 || (pq_bits == 6 && pq_dim == 48);
}

// How many pairs of a cluster share a workgroup (0: the group kernel does not apply).  It serves 8-bit and 4-bit
// codes in 16-byte chunks, 5- to 7-bit codes of 32 to 96 sub-spaces, sub-vectors of 1, 2 or 4 components and fixed
// encoding constants.  The widest layout
// is taken that leaves room for 16 waves per compute unit (scan_group_threads: 40 KB of LDS with four waves, 80 KB with eight),
// but not four pairs on eight waves where two pairs leave room for more than 16 waves (five workgroups of 32 KB).  Eight
// waves pay where the shared table build is heavy: half tables at four pairs with sub-vectors of four components (two components, 32
// sub-spaces: two pairs 1.00 ms, four 1.04*), the others from two components on (one was not measured).
// Measured, whole search of 10^6 vectors, 10,000 queries and 20 probes, 8-bit codes (one pair / two / four, the figure of eight waves marked *):
//   e5m3  32 sub-spaces 1.35 (two) / 1.22 (four); 48: 1.23 (two) / 1.33* (four); 64: 1.69 (two) / 1.64* (four)
//   half  32 sub-spaces 1.39 (two) / 1.32* (four); 48: 1.58 / 1.47* / 1.97; 64: 2.48 / 1.92* / 2.17
//   float 32 sub-spaces 2.27 / 1.68* / 2.14; 48: 2.11 / 2.24 / -; 64: 3.00 / 2.88 / - (one workgroup per compute unit: left with one pair);
//         16: 0.91 / 0.79 / 0.99* (hence no four pairs of float tables with 8-bit codes)
// and 64 probes of 2,000 vectors, 32 sub-spaces: e5m3 3.03 / 2.62, half 3.20 / 3.02* (two / four), float 5.36 / 4.01* (one / two).
// With 4-bit codes (16-entry rows, a few KB of tables) four pairs for every dtype: filtered scan, 10^8 vectors,
// 64 sub-spaces, e5m3 6.67 / 5.95 / 5.21 ms, half 7.56 / 6.48 / 4.62, float 6.31 / 4.71 / 4.02.  Bit-packed codes, whole
// search of 10^6 vectors, 20 probes: 7 bits e5m3 2.35 / 1.67 / 1.46 ms, half 2.45 / 1.90 / -; 6 bits 1.91 / 1.59 / 1.37, half
// 1.98 / 1.76, float 1.97 / 1.37; 5 bits 2.03 / 1.58 / 1.37, half 2.09 / 1.72, float 1.74 / 1.23 (64 sub-spaces).
// Other numbers of them, e5m3 one / two / four pairs, half and float one / two:
//   32  7 bits 2.03 / 1.28 / 1.09, 2.21 / 1.40, 2.48 / 1.20; 6 bits 1.33 / 1.18 / 1.01, 1.40 / 1.28, 1.30 / 1.07;
//       5 bits 1.87 / 1.11 / 0.95, 1.94 / 1.20, 1.61 / 0.97
//   48  6 bits 1.08 / 1.03 / 0.93, 1.14 / 1.12, 1.06 / 0.93
//   96  (one component) 7 bits 1.78 / 1.42 / 1.47, 2.21 / 1.94*, 2.69 / 2.50*; 6 bits 1.62 / 1.35 / 1.23, 1.72 / 1.51,
//       1.93 / 1.46*; 5 bits 1.52 / 1.29 / 1.16, 1.58 / 1.42, 1.32 / 1.08
// (Four pairs of their wider tables and the split scan of one pair are not built.  One kernel per width that walks any
// number of sub-spaces in units of 32 costs 64 of them 8 to 12 %: the unit's place joins every address and the walk's
// state spills.)
int scan_group_width(const ivfpq_index* idx, int lut_dtype, const Fp8Mode& fp8, uint32_t order_block) {
    const bool packed = idx->pq_bits != 8 && idx->pq_bits != 4;
    if (fp8.per_table || (packed ? !scan_group_packed(idx->pq_bits, idx->pq_dim) : chunk_width(idx) != 16)) return 0;
    if (idx->pq_bits == 4 && idx->pq_dim % 16 != 0) return 0;      // the table is built in blocks of 256 entries
    const int m = idx->d / idx->pq_dim;
    if (m != 1 && m != 2 && m != 4) return 0;
    const int want = idx->tuning.scan_share;
    if (want == 1) return 0;
    const bool one_byte = lut_dtype == IVFPQ_LUT_FP8_E5M3 || lut_dtype == IVFPQ_LUT_FP8_E4M4;
    for (int G : {4, 2}) {
        if (want != 0 && want != G) continue;
        if (order_block < (uint32_t)G || order_block % (uint32_t)G) continue;
        if (packed && G == 4 && !one_byte) continue;
        const int threads = scan_group_threads(idx, lut_dtype, G);
        const size_t lds = scan_group_lds_bytes(idx, lut_dtype, G, threads);
        if (want == G) { if (lds <= kLdsBytes) return G; continue; }
        if (lds > (threads >= 512 ? kGroupLds2 : kGroupLds4)) continue;
        if (idx->pq_bits == 8 && G == 4 && lut_dtype == IVFPQ_LUT_FP32) continue;
        if (threads == 512 && m < (G == 4 && !one_byte ? 4 : 2)) continue;
        if (G == 4 && lds > kGroupLds4 && scan_group_lds_bytes(idx, lut_dtype, 2, 256) <= kLdsBytes / 5) continue;
        return G;
    }
    return 0;
}
int launch_scan_group(const ivfpq_index* idx, const ScanArgs& a, int lut_dtype, int G, hipStream_t st) {
    const int threads = scan_group_threads(idx, lut_dtype, G);
    const size_t lds = scan_group_lds_bytes(idx, lut_dtype, G, threads);
    if (lds > kLdsBytes) return fail(IVFPQ_EUNSUPPORTED, "tables + staging + pad need %zu bytes of LDS (limit %zu)", lds, kLdsBytes);
    switch (lut_dtype) {
        case IVFPQ_LUT_FP32: return launch_scan_group_kernel<IVFPQ_LUT_FP32>(a, G, threads, lds, st);
        case IVFPQ_LUT_FP16: return launch_scan_group_kernel<IVFPQ_LUT_FP16>(a, G, threads, lds, st);
        case IVFPQ_LUT_FP8_E5M3: return launch_scan_group_kernel<IVFPQ_LUT_FP8_E5M3>(a, G, threads, lds, st);
        default: return launch_scan_group_kernel<IVFPQ_LUT_FP8_E4M4>(a, G, threads, lds, st);
    }
}

// Pairs a workgroup of the group kernel takes for the queries' nearest probes, or 0 where scan_kernel takes a query each (the line and both of
// its sides: nearest_by_groups).
int nearest_group_width(const ivfpq_index* idx, int lut_dtype, const Fp8Mode& fp8, int nq, int k) {
    const ivfpq::Tuning& t = idx->tuning;
    if (t.scan_route != 0 || t.scan_share != 0 || t.order_block != 0 || t.scan_threads != 0 || t.lds_pad != 0) return 0;
    const int G = scan_group_width(idx, lut_dtype, fp8, kOrderBlock);
    if (G == 0) return 0;
    const bool eight_waves = scan_group_lds_bytes(idx, lut_dtype, G, scan_group_threads(idx, lut_dtype, G)) > kGroupLds4;
    return ivfpq::nearest_by_groups({nq, k, idx->n, idx->list_mean, idx->list_typical, (double)idx->sorted_padded_sizes[0], idx->pq_bits, idx->pq_dim,
                                     (int)lut_elem_bytes(lut_dtype), G, eight_waves}) ? G : 0;
}

// A grid that leaves wave slots of the chip empty takes larger workgroups: tables are built and lists walked by more
// waves at once (filtered scan of one query, 19 pairs: 21.6 -> 9 us with 1024 threads instead of 256).
int scan_threads_of_grid(const ivfpq_index* idx, int lut_dtype, size_t blocks) {
    int threads = scan_threads(idx, lut_dtype);
    if (!idx->tuning.scan_threads)
        while (threads < 1024 && blocks * (threads / 64) < kWaveSlots &&
               scan_lds_bytes_staged(idx, lut_dtype, threads * 2) <= kLdsBytes) threads *= 2;
    return threads;
}
int launch_scan(const ivfpq_index* idx, ScanArgs a, int lut_dtype, dim3 grid, hipStream_t st) {
    const int threads = scan_threads_of_grid(idx, lut_dtype, grid.x);
    const size_t lds = std::max(scan_lds_bytes_staged(idx, lut_dtype, threads), a.mode == 1 && a.k_bound > 0 ? kBoundLds : (size_t)0);
    if (lds > kLdsBytes)
        return fail(IVFPQ_EUNSUPPORTED, "lookup table + residual + staging need %zu bytes of LDS (limit %zu)", lds, kLdsBytes);
    const int cw = chunk_width(idx);
    const int nch = idx->code_bytes() / cw;
    a.n_chunks = nch;
    const int bits = idx->pq_bits;
    switch (lut_dtype) {
        case IVFPQ_LUT_FP32: return launch_scan_lut<IVFPQ_LUT_FP32>(a, bits, cw, nch, grid, threads, lds, st);
        case IVFPQ_LUT_FP16: return launch_scan_lut<IVFPQ_LUT_FP16>(a, bits, cw, nch, grid, threads, lds, st);
        case IVFPQ_LUT_FP8_E5M3: return launch_scan_lut<IVFPQ_LUT_FP8_E5M3>(a, bits, cw, nch, grid, threads, lds, st);
        default: return launch_scan_lut<IVFPQ_LUT_FP8_E4M4>(a, bits, cw, nch, grid, threads, lds, st);
    }
}

Fp8Mode fp8_mode(const ivfpq_index* idx, int lut_dtype) {
    Fp8Mode m{};
    if (lut_dtype == IVFPQ_LUT_FP8_E5M3 || lut_dtype == IVFPQ_LUT_FP8_E4M4) {
        const ivfpq::Fp8Options& o = idx->fp8_opt[lut_dtype - IVFPQ_LUT_FP8_E5M3];
        m.fixed = fp8_params(lut_dtype == IVFPQ_LUT_FP8_E5M3 ? Fp8Format<IVFPQ_LUT_FP8_E5M3>::shift : Fp8Format<IVFPQ_LUT_FP8_E4M4>::shift,
                             o.bias, o.truncate);
        m.truncate = o.truncate;
        m.per_table = o.per_table;
    }
    return m;
}

ScanArgs base_scan_args(const ivfpq_index* idx, int lut_dtype) {
    ScanArgs a{};
    a.centroids = idx->dev.centroids;
    a.codebooks = idx->dev.codebooks;
    a.list_sizes = idx->dev.list_sizes;
    a.group_offsets = idx->dev.group_offsets;
    a.codes = idx->dev.codes;
    a.d = idx->d; a.pq_dim = idx->pq_dim; a.m = idx->m(); a.bits = idx->pq_bits;
    a.n_lists = idx->n_lists;
    a.fp8 = fp8_mode(idx, lut_dtype);
    a.single_list = -1;
    a.early_exit = idx->tuning.early_exit >= 0;
    return a;
}

// ---- the matrix-core filter: for the grouped route, unless a knob asks for the table kernels ----
// Tables that saturate below (2 x the largest codeword)^2 hide so much of far vectors' distances that most pass, and a listed
// vector costs several table lookups' worth (e4m4 of 31,744 against codewords of 100 and more, 17 M vectors looked up: 351 us, table kernels
// 164).
float table_top(int lut_dtype, const Fp8Mode& fp8) {
    float top = __builtin_inff();
    if (lut_dtype == IVFPQ_LUT_FP16) top = 65504.f;
    else if (lut_dtype != IVFPQ_LUT_FP32) std::memcpy(&top, &fp8.fixed.hi, 4);
    return top;
}
bool filter_applies(const ivfpq_index* idx, int lut_dtype, const Fp8Mode& fp8) {
    const ivfpq::Tuning& t = idx->tuning;
    if (!(4.f * idx->word_norm_max * idx->word_norm_max <= table_top(lut_dtype, fp8))) return false;
    return t.early_exit >= 0 && t.scan_share == 0 && t.order_block == 0 && t.scan_threads == 0 && t.lds_pad == 0 && !fp8.per_table &&
           idx->word_norm_max >= 0.f && filter_supported(idx->pq_bits, idx->pq_dim, idx->d, chunk_width(idx));
}
// By the number of vectors that are looked up, as scan_route, and by k against the length of a list: the bound is the k-th of one list.
// The filter has a cost of its own (codebooks that two kernels load); us a search, the better table route / filter:
//   k / length 0.01  6 M 75 / 64, 75 / 77, 84 / 81, 68 / 71, 93 / 72, 82 / 78; 9 M 91 / 64, 91 / 81, 102 / 92, 82 / 83, 121 / 91, 125 / 85
//              0.05  6 M 80 / 76, 90 / 88, 83 / 92; 9 M 97 / 75, 108 / 96, 97 / 107; 12 M 118 / 89, 132 / 107, 108 / 110
//              0.1   6 M 92 / 97, 96 / 125, 97 / 95, 145 / 122; 12 M 134 / 116, 142 / 160, 140 / 113, 237 / 164; 30 M 270 / 144, 244 / 206
// (200,000 unit-norm rows in 200 lists, 60 and 20 probes; 10^6 in 1,024, 20; 200,000 of 128 components in 100, 30, where 0.05; 100,000 in
// 100, 30, where 0.01 and 0.1; 10^6 in 555, 4-bit codes, 30).
// Of larger batches the cheaper side by what either spends, in listed vectors (25 to 45 ps each): the tables `pair` for a pair's table and
// `vector` for a vector looked up; the filter one for each vector that it lists, whose share the upload sampled (pass_share; one-byte
// tables, whose rounding widens the limit, list more), and `block` for a vector of a list and each 64 of the list's pairs, however
// few of a block there are.  Fitted to 3,081 searches: 10^6 to 10^8 vectors in lists of 500 to 3,300 and of 1 to 1,000 Gaussian components, 1 to 2,000
// pairs a list, k / length 0.005 to 0.8, every code length and table.  The side taken is 0.4 % slower than the better one in the
// mean, 1.7 % of the searches lose more than a tenth, the worst takes 1.75 times as long.  Some of them, us, tables / filter, by the sampled share:
//   10^8 vectors in 50,000 lists, 64 probes, 10,000 queries (13 pairs a list), 32-byte codes   e5m3 0.021 4,980 / 4,831, 0.048 5,284 / 7,279;
//                  half 0.008 5,814 / 4,111, 0.017 6,165 / 5,198, 0.087 6,982 / 9,633; float 0.017 7,839 / 5,084, 0.086 8,442 / 9,489
//                  64 codes of 4 bits e5m3 0.019 5,768 / 5,746, 0.061 5,972 / 8,017; half 0.008 4,579 / 4,999, 0.022 4,774 / 5,888
//   the same, 20 probes (4 pairs a list), 32-byte codes   e5m3 0.039 2,425 / 3,006; half 0.015 2,820 / 2,599, 0.033 3,036 / 3,869
//   10^7 in 5,000 (126 pairs a list)    e5m3 0.009 3,450 / 1,629, 0.024 3,655 / 2,599;  in 20,000 (32)  0.087 2,767 / 1,912, 0.285 3,215 / 4,496
struct FilterCost {
    double pair, vector, block;
};
FilterCost filter_cost(int bits, int pq_dim, int table_bytes, bool one_pair) {
    if (one_pair) {                     // tables too large for two pairs, or codes not in 16-byte pieces
        if (bits == 4) return table_bytes == 1 ? FilterCost{42, 0.088, 0.2} : table_bytes == 2 ? FilterCost{65, 0.14, 0.1} : FilterCost{74, 0.17, 0.1};
        return FilterCost{100, 0.14 + 0.0024 * pq_dim, 0.4};
    }
    if (bits == 8)
        return table_bytes == 1 ? FilterCost{45, 0.001 * pq_dim, 0.25}
             : table_bytes == 2 ? FilterCost{110, 0.002 * pq_dim - 0.02, 0.4} : FilterCost{95, 0.0032 * pq_dim - 0.02, 0.44};
    if (bits == 4) {
        if (table_bytes == 1) return FilterCost{57, 0.00054 * pq_dim, 0.4};
        // (float tables of 32 4-bit codes: the table kernel takes five times as long as with 64)
        return table_bytes == 4 && pq_dim < 64 ? FilterCost{50, 0.25, 0.5} : FilterCost{24, 0.027, 0.5};
    }
    const FilterCost c = table_bytes == 1 ? FilterCost{20, 0.078, 0.4} : table_bytes == 2 ? FilterCost{60, 0.2, 0.4}
                       : bits == 7 ? FilterCost{60, 0.18, 0.4} : FilterCost{50, 0.1, 0.4};
    return FilterCost{c.pair, c.vector * pq_dim / 64.0, c.block};
}
bool filter_pays(const ivfpq_index* idx, int lut_dtype, const Fp8Mode& fp8, int nq, int n_probes, int k) {
    if (idx->tuning.scan_route != 0) return true;
    const double length = (double)idx->n / (double)idx->n_lists, share = (double)k / length, pairs = (double)nq * (n_probes - 1);
    if (!(pairs * length >= kFilterLookups + 1e8 * share) || idx->pass_shares.ranks == 0) return false;
    const FilterCost c = filter_cost(idx->pq_bits, idx->pq_dim, lut_elem_bytes(lut_dtype), scan_group_width(idx, lut_dtype, fp8, kOrderBlock) == 0);
    // blocks a pair: of few pairs a list, some lists have none; of many, half a block more than is full
    const double per_list = pairs / (double)idx->n_lists;
    const double blocks = per_list < 20 ? (1.0 - std::exp(-per_list)) / per_list : std::min(1.0 / per_list, 1.0 / kFilterPairs + 0.5 / per_list);
    const double most = std::min(0.5, c.pair / length + c.vector - c.block * blocks);       // (nothing was measured of shorter lists)
    const double wider = 1.0 / (1.0 - stored_loss(lut_dtype, fp8.truncate)) - 1.0 + 0.012;            // of the limit against the bound; the rest is eta's
    return pass_share(idx->pass_shares, n_probes, share, wider) <= most;
}
void filter_constants(const ivfpq_index* idx, int lut_dtype, const Fp8Mode& fp8, FilterArgs* a) {
    const FilterBound bound = filter_bound(lut_dtype, fp8.truncate, idx->pq_dim, idx->d);
    a->scale = bound.scale;
    a->add = bound.add;
    a->eta = bound.eta;
    a->top = table_top(lut_dtype, fp8);
    a->word_norm_max = idx->word_norm_max;
    a->fp8 = fp8.fixed;
    a->truncate = fp8.truncate;
}
int launch_candidates(const FilterArgs& a, int lut_dtype, hipStream_t st) {
    switch (lut_dtype) {
        case IVFPQ_LUT_FP32: return launch_candidates_lut<IVFPQ_LUT_FP32>(a, st);
        case IVFPQ_LUT_FP16: return launch_candidates_lut<IVFPQ_LUT_FP16>(a, st);
        case IVFPQ_LUT_FP8_E5M3: return launch_candidates_lut<IVFPQ_LUT_FP8_E5M3>(a, st);
        default: return launch_candidates_lut<IVFPQ_LUT_FP8_E4M4>(a, st);
    }
}

// ---- what ivfpq_scan_kernel_info says of a launch ----
const char* const kLutNames[4] = {"fp32", "fp16", "e5m3", "e4m4"};
void describe_filter(const ivfpq_index* idx, int lut_dtype, char* buf, size_t bytes) {
    snprintf(buf, bytes, "scan_filter_kernel<%d-bit codes, %d components a sub-space, d = %d> and candidate_kernel<%s>, %zu and %zu bytes of LDS",
             idx->pq_bits, idx->m(), idx->d, kLutNames[lut_dtype], filter_lds_bytes(idx->pq_bits, idx->d), candidate_lds_bytes(idx->pq_bits, idx->d));
}
void describe_group(const ivfpq_index* idx, int lut_dtype, int G, char* buf, size_t bytes) {
    const int threads = scan_group_threads(idx, lut_dtype, G);
    snprintf(buf, bytes, "scan_group_kernel<%s, %d-bit codes, %d chunks, %d pairs> %d threads, %zu bytes of LDS", kLutNames[lut_dtype], idx->pq_bits,
             idx->code_bytes() / chunk_width(idx), G, threads, scan_group_lds_bytes(idx, lut_dtype, G, threads));
}
void describe_scan(const ivfpq_index* idx, int lut_dtype, int threads, char* buf, size_t bytes) {
    const int cw = chunk_width(idx), nch = idx->code_bytes() / cw;
    snprintf(buf, bytes, "scan_kernel<%s, %d-bit codes, %d-byte chunks x %d> %d threads, %zu bytes of LDS", kLutNames[lut_dtype],
             idx->pq_bits, cw, cw == 16 ? nch : 0, threads, scan_lds_bytes_staged(idx, lut_dtype, threads));
}

// ---- stage timing ----
int timing_mark(const ivfpq_index* idx, hipStream_t st, void** out) {
    if (idx->events_used == idx->event_pool.size()) {
        hipEvent_t e;
        HIP_TRY(hipEventCreate(&e));
        idx->event_pool.push_back((void*)e);
    }
    hipEvent_t e = (hipEvent_t)idx->event_pool[idx->events_used++];
    HIP_TRY(hipEventRecord(e, st));
    *out = (void*)e;
    return IVFPQ_OK;
}

struct StageTimer {
    const ivfpq_index* idx; hipStream_t st; int stage; void* a = nullptr; bool on;
    StageTimer(const ivfpq_index* i, hipStream_t s, int stage_) : idx(i), st(s), stage(stage_), on(i->timing) {}
    int begin() { return on ? timing_mark(idx, st, &a) : IVFPQ_OK; }
    int end() {
        if (!on) return IVFPQ_OK;
        void* b = nullptr;
        if (int s = timing_mark(idx, st, &b)) return s;
        idx->spans.push_back({a, b, stage, 1.f});
        return IVFPQ_OK;
    }
    // the span just ended covers the work of `other` as well: that stage gets all of it but `share`
    void divide(int other, float share) {
        if (!on) return;
        auto& own = idx->spans.back();
        own.share = share;
        const auto rest = ivfpq_index::Span{own.a, own.b, other, 1.f - share};
        idx->spans.push_back(rest);
    }
};

// static_scratch: the workspace is the library's own fixed device array (d_ws is resolved after the checks)
int search_impl(const ivfpq_index* idx, const float* d_queries, int64_t nq, const uint32_t* d_probes_in,
                int32_t n_probes, int32_t k, int32_t lut_dtype, int64_t* d_ids, float* d_dists,
                void* d_ws, size_t ws_bytes, void* hip_stream, bool static_scratch = false) {
    if (int s = check_search_args(idx, d_queries, nq, n_probes, k, lut_dtype, true)) return s;
    if (nq > 0 && (!d_ids || !d_dists)) return fail(IVFPQ_EINVAL, "null output pointer");
    Plan plan;
    if (static_scratch) {
        // sized before anything touches the device: a request beyond the fixed array is refused as such
        if (int s = make_plan(idx, nq, n_probes, d_probes_in != nullptr, &plan, kStaticScratchBytes)) return s;
        if (plan.total > kStaticScratchBytes)
            return fail(IVFPQ_ENOSPACE, "one query with %d probes on this index needs %zu bytes of scratch; the static "
                        "scratch holds %zu (use ivfpq_search with a caller workspace)", n_probes, plan.total, kStaticScratchBytes);
    }
    if (int s = check_device(idx)) return s;
    if (nq == 0) return IVFPQ_OK;
    if (static_scratch) {
        if (int s = static_scratch_ptr(&d_ws)) return s;
        ws_bytes = kStaticScratchBytes;
    } else if (int s = make_plan(idx, nq, n_probes, d_probes_in != nullptr, &plan)) {
        return s;
    }
    if (!d_ws || ws_bytes < plan.total)
        return fail(IVFPQ_ENOSPACE, "workspace of %zu bytes given, %zu needed", ws_bytes, plan.total);
    if (scan_lds_bytes_staged(idx, lut_dtype, scan_threads(idx, lut_dtype)) > kLdsBytes)
        return fail(IVFPQ_EUNSUPPORTED, "lookup table + residual + staging need %zu bytes of LDS (limit %zu)",
                    scan_lds_bytes_staged(idx, lut_dtype, scan_threads(idx, lut_dtype)), kLdsBytes);
    hipStream_t st = (hipStream_t)hip_stream;
    unsigned char* ws = (unsigned char*)d_ws;
    uint32_t* w_probes = (uint32_t*)(ws + plan.probes);
    float* w_probe_d = (float*)(ws + plan.probe_d);
    uint32_t* w_roff = (uint32_t*)(ws + plan.roff);
    uint4* w_pairs = (uint4*)(ws + plan.pairs);
    uint32_t* w_bounds = (uint32_t*)(ws + plan.bounds);
    uint32_t* w_counts = (uint32_t*)(ws + plan.counts);
    uint32_t* w_Rpos = (uint32_t*)(ws + plan.Rpos);
    float* w_D = (float*)(ws + plan.D);
    StripSummary* w_S = (StripSummary*)(ws + plan.S);
    float* w_R = (float*)(ws + plan.R);

    if (idx->timing) { idx->events_used = 0; idx->spans.clear(); idx->stage_valid = true; idx->scan_kernel_lut = -1; }
    StageTimer whole(idx, st, 3);
    if (int s = whole.begin()) return s;
    for (int64_t q0 = 0; q0 < nq; q0 += plan.tile) {
        const int tq = (int)std::min<int64_t>(plan.tile, nq - q0);
        const float* qt = d_queries + (size_t)q0 * idx->d;
        // step 1
        StageTimer t0(idx, st, 0);
        if (int s = t0.begin()) return s;
        if (!d_probes_in) {
            StripSummary* strips = w_S;
            bool exact = false;
            StageTimer t4(idx, st, 4);
            if (int s = t4.begin()) return s;
            if (int s = launch_step_1a(idx, qt, tq, n_probes, (uint32_t*)w_D, &strips, &exact, ws + plan.split, st)) return s;
            if (int s = t4.end()) return s;
            launch_select_probes((int)tq, exact, st, (uint32_t*)w_D, (const StripSummary*)strips,
                                 coarse_strip_width(tq, idx->n_lists), qt,
                                 idx->dev.centroids, idx->centroid_norm_max, idx->rank_crowd, idx->d, idx->n_lists,
                                 n_probes, idx->dev.list_sizes, idx->dev.group_offsets, w_probes, w_probe_d, w_roff, w_pairs, k, w_counts);
            HIP_TRY(hipGetLastError());
        } else {
            hipLaunchKernelGGL(layout_probes_kernel, dim3((tq + 255) / 256), dim3(256), 0, st,
                               d_probes_in + (size_t)q0 * n_probes, tq, n_probes, idx->n_lists, idx->dev.list_sizes,
                               idx->dev.group_offsets, w_probes, w_roff, w_pairs);
            HIP_TRY(hipGetLastError());
        }
        if (int s = t0.end()) return s;
        // steps 2-4
        StageTimer t1(idx, st, 1);
        if (int s = t1.begin()) return s;
        // nearest probe of every query first: its R values give the bound that filters the rest (little work: all probes at once)
        ScanArgs a = base_scan_args(idx, lut_dtype);
        a.queries = qt; a.pairs = w_pairs; a.R = w_R; a.stride = plan.stride;
        a.n_probes = n_probes; a.bounds = w_bounds; a.counts = w_counts; a.Rpos = w_Rpos;
        const ScanRoute route = scan_route(idx, tq, n_probes);
        const bool whole_rows = route == ScanRoute::kWholeRows;
        // how the others follow: their grouping and the filter's lists, whose counters the first launch clears
        const size_t n_pairs = (size_t)tq * (n_probes - 1);
        const bool grouped = n_probes > 1 && route == ScanRoute::kGrouped && group_pairs_by_cluster(n_pairs);
        // The filter's lists take the place of the ranking values, which nothing reads any more (a search with given probes has none).
        FilterLists lists = filter_lists(idx, (size_t)tq, n_probes, filter_item_vectors(idx, n_pairs));
        while (lists.bytes > plan.R - plan.D && lists.per_item < (uint32_t)kFilterVectors) lists = filter_lists(idx, (size_t)tq, n_probes, lists.per_item * 2);
        const bool filter = grouped && filter_applies(idx, lut_dtype, a.fp8) && filter_pays(idx, lut_dtype, a.fp8, tq, n_probes, k) && ((uintptr_t)qt & 7) == 0 &&
                            lists.max_items < ((size_t)1 << 31) && lists.bytes <= plan.R - plan.D;
        uint32_t* w_starts = filter ? (uint32_t*)(ws + plan.D) : nullptr;
        uint32_t* w_lc = (uint32_t*)(ws + plan.list_counts);         // counts and cursors are neighbours in the plan
        a.mode = whole_rows ? 3 : 1;
        if (n_probes > 1 && !whole_rows) {
            a.k_bound = k;
            a.starts = w_starts;
            if (grouped) { a.clear[0] = w_lc; a.n_clear[0] = (uint32_t)((plan.list_offsets - plan.list_counts) / 4); }
            if (filter) { a.clear[1] = (uint32_t*)(ws + plan.D + lists.totals); a.n_clear[1] = 2u; }
        }
        // a timed search notes what its first tile launches for the probes other than the nearest
        auto note = [&](auto describe, auto... what) {
            if (!idx->timing || idx->scan_kernel_lut >= 0) return;
            describe(idx, lut_dtype, what..., idx->scan_kernel, sizeof idx->scan_kernel);
            idx->scan_kernel_lut = lut_dtype;
        };
        auto note_scan = [&](size_t blocks) { if (idx->timing) note(describe_scan, scan_threads_of_grid(idx, lut_dtype, blocks)); };
        StageTimer t5(idx, st, 5);
        StageTimer t6(idx, st, 6);
        if (int s = t5.begin()) return s;
        if (const int G = grouped && !d_probes_in ? nearest_group_width(idx, lut_dtype, a.fp8, tq, k) : 0) {
            // the selection has left the nearest clusters in w_counts; the other probes' order comes later
            uint32_t* w_near = (uint32_t*)(ws + plan.order);
            hipLaunchKernelGGL(nearest_order_kernel, dim3((idx->n_lists + kWave - 1) / kWave), dim3(1024), 0, st, w_counts, tq, w_near);
            HIP_TRY(hipGetLastError());
            ScanArgs near = a;
            near.order = w_near;
            near.n_pairs = (uint32_t)tq;
            near.order_block = kOrderBlock;
            near.n_chunks = idx->code_bytes() / chunk_width(idx);
            if (int s = launch_scan_group(idx, near, lut_dtype, G, st)) return s;
            StageTimer t7(idx, st, 7);
            if (int s = t7.begin()) return s;
            hipLaunchKernelGGL(bound_wave_kernel, dim3((unsigned)((tq + kBoundQueries - 1) / kBoundQueries)), dim3(64 * kBoundQueries), 0, st, near, tq);
            HIP_TRY(hipGetLastError());
            if (int s = t7.end()) return s;
        } else if (int s = launch_scan(idx, a, lut_dtype, dim3((unsigned)((size_t)tq * (whole_rows ? n_probes : 1))), st)) {
            return s;
        }
        if (int s = t5.end()) return s;
        if (whole_rows && n_probes > 1) note_scan((size_t)tq * n_probes);
        if (whole_rows) t5.divide(6, 1.f / (float)n_probes);      // one launch does the work of both: divided by their pairs
        if (n_probes > 1 && !whole_rows) {
            a.mode = 2;
            if (grouped) {
                uint32_t* w_order = (uint32_t*)(ws + plan.order);
                uint32_t* w_cur = (uint32_t*)(ws + plan.list_cursor);
                uint32_t* w_lo = (uint32_t*)(ws + plan.list_offsets);
                const unsigned pb = (unsigned)((n_pairs + 255) / 256);
                uint32_t* w_totals = (uint32_t*)(ws + plan.D + lists.totals);
                uint4* w_items = (uint4*)(ws + plan.D + lists.items);
                FilterArgs f{};
                if (filter) filter_constants(idx, lut_dtype, a.fp8, &f);
                const PairCull cull{filter ? w_probe_d : nullptr, w_bounds, idx->dev.list_radii, f.scale, f.add, f.top};
                const PairRecords records{filter ? (uint4*)(ws + plan.D + lists.records) : nullptr, w_probe_d, w_bounds};
                // the place of every cluster's pairs; with the filter also its work items
                auto offsets = [&] {
                    if (filter)
                        hipLaunchKernelGGL(filter_items_kernel, dim3((idx->n_lists + kWave - 1) / kWave), dim3(1024), 0, st, w_lc, idx->dev.list_sizes,
                                           idx->dev.group_offsets, idx->n_lists, lists.per_item, w_lo, w_totals, w_items, (uint32_t)lists.max_items);
                    else
                        hipLaunchKernelGGL(pair_offsets_kernel, dim3(1), dim3(1024), 0, st, w_lc, idx->n_lists, w_lo);
                };
                if (idx->n_lists <= kPairLdsLists) {
                    const uint32_t chunk = pair_chunk(n_pairs);
                    const unsigned cb = (unsigned)((n_pairs + chunk - 1) / chunk);
                    const size_t lds = (size_t)idx->n_lists * 4;
                    if (int s = allow_full_lds(pair_scatter_lds_kernel)) return s;
                    hipLaunchKernelGGL(pair_count_lds_kernel, dim3(cb), dim3(1024), lds, st, w_pairs, (uint32_t)n_pairs, chunk, n_probes, idx->n_lists, w_lc, cull);
                    offsets();
                    hipLaunchKernelGGL(pair_scatter_lds_kernel, dim3(cb), dim3(1024), 2 * lds, st, w_pairs, (uint32_t)n_pairs, chunk, n_probes,
                                       idx->n_lists, w_lo, w_cur, w_order, records, cull);
                } else {
                    hipLaunchKernelGGL(pair_count_kernel, dim3(pb), dim3(256), 0, st, w_pairs, (uint32_t)n_pairs, n_probes, idx->n_lists, w_lc, cull);
                    offsets();
                    hipLaunchKernelGGL(pair_scatter_kernel, dim3(pb), dim3(256), 0, st, w_pairs, (uint32_t)n_pairs, n_probes, idx->n_lists,
                                       w_lo, w_cur, w_order, records, cull);
                }
                HIP_TRY(hipGetLastError());
                a.order = w_order;
                a.n_pairs = (uint32_t)n_pairs;
                const uint32_t blk = idx->tuning.order_block > 0 ? (uint32_t)idx->tuning.order_block : kOrderBlock;
                a.order_block = blk;
                if (int s = t6.begin()) return s;
                if (filter) {
                    f.queries = qt; f.centroids = a.centroids; f.codebooks = a.codebooks; f.codes = a.codes;
                    f.pairs = w_pairs; f.bounds = w_bounds; f.starts = w_starts; f.counts = w_counts;
                    f.row_key = (uint32_t*)w_R; f.row_pos = w_Rpos; f.stride = plan.stride;
                    f.records = records.records; f.items = w_items; f.n_items = w_totals + 1;
                    f.nq = tq; f.n_probes = n_probes;
                    f.d = idx->d; f.pq_dim = idx->pq_dim; f.m = idx->m(); f.bits = idx->pq_bits;
                    f.code_bytes = idx->code_bytes(); f.chunk_width = chunk_width(idx);
                    note(describe_filter);
                    if (int s = launch_filter(f, st)) return s;
                    if (int s = launch_candidates(f, lut_dtype, st)) return s;
                } else if (const int G = scan_group_width(idx, lut_dtype, a.fp8, blk)) {
                    a.n_chunks = idx->code_bytes() / chunk_width(idx);
                    note(describe_group, G);
                    if (int s = launch_scan_group(idx, a, lut_dtype, G, st)) return s;
                } else {
                    const size_t grid = (n_pairs + 8 * (size_t)blk - 1) / (8 * (size_t)blk) * (8 * (size_t)blk);
                    note_scan(grid);
                    if (int s = launch_scan(idx, a, lut_dtype, dim3((unsigned)grid), st)) return s;
                }
            } else {
                if (int s = t6.begin()) return s;
                note_scan(n_pairs);
                if (int s = launch_scan(idx, a, lut_dtype, dim3((unsigned)n_pairs), st)) return s;
            }
            if (int s = t6.end()) return s;
        }
        if (int s = t1.end()) return s;
        // step 5
        StageTimer t2(idx, st, 2);
        if (int s = t2.begin()) return s;
        auto topk = [&](auto kernel, int threads) {
            hipLaunchKernelGGL(kernel, dim3(tq), dim3(threads), 0, st, w_R, w_Rpos, plan.stride, w_roff, w_probes, w_bounds, w_counts,
                               n_probes, idx->n_lists, k, idx->dev.list_offsets, idx->dev.ids, d_ids + (size_t)q0 * k, d_dists + (size_t)q0 * k,
                               n_probes > 1 && !whole_rows);
        };
        if (tq <= kFewQueries) topk(topk_kernel<SEL_CAP, 1024>, 1024);
        else if (k <= SEL_CAP_SMALL) topk(topk_kernel<SEL_CAP_SMALL, SEL_THREADS>, SEL_THREADS);
        else topk(topk_kernel<SEL_CAP, SEL_THREADS>, SEL_THREADS);
        HIP_TRY(hipGetLastError());
        if (int s = t2.end()) return s;
    }
    if (int s = whole.end()) return s;
    return IVFPQ_OK;
}

}  // namespace

namespace ivfpq {
void release_device_state(ivfpq_index* idx) {
    for (void* e : idx->event_pool) (void)hipEventDestroy((hipEvent_t)e);
    idx->event_pool.clear();
}
}  // namespace ivfpq

extern "C" {

size_t ivfpq_device_bytes(const ivfpq_index_t* index) {
    if (!index) { set_error("ivfpq_device_bytes: null index"); return 0; }
    return image_layout(index).total;
}

}  // extern "C"

namespace {
// Codes in list order (vectors v0 ... of the index, code_bytes each) to their places in the interleaved layout, for groups
// [g0, g1): one wave per group of 64 vectors; lanes past the end of a cluster write zeros.  W: one chunk.
// Bound by the host link the codes arrive over (48 MB: 1.7 ms); the rearrangement on 16 host threads, into a cleared
// buffer that was then copied, took 10 ms.
template <class W>
__global__ void __launch_bounds__(256)
interleave_codes_kernel(const W* __restrict__ raw, int64_t v0, const int64_t* __restrict__ list_offsets,
                        const int64_t* __restrict__ group_offsets, int n_lists, int64_t g0, int64_t g1, int n_chunks, W* __restrict__ codes) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t g = g0 + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= g1) return;
    int lo = 0, hi = n_lists;                          // the last list that starts at or before group g (empty ones start there too)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (group_offsets[mid] <= g) lo = mid; else hi = mid;
    }
    const int64_t v = list_offsets[lo] + (g - group_offsets[lo]) * 64 + lane;
    const bool ok = v < list_offsets[lo + 1];
    for (int c = 0; c < n_chunks; ++c) {
        W w{};
        if (ok) w = raw[(v - v0) * n_chunks + c];
        codes[(g * n_chunks + c) * 64 + lane] = w;
    }
}

// The largest squared norm of a decoded residual of every cluster, as the bits of a float, from the squared norms of the codewords
// (in the LDS where they fit).  One wave per run of 64-vector groups; bound by the LDS reads, one per code (10^6 vectors of 48
// codes: 15 us).
__global__ void __launch_bounds__(1024)
list_radii_kernel(const unsigned char* __restrict__ codes, const float* __restrict__ word_norms, const int64_t* __restrict__ list_offsets,
                  const int64_t* __restrict__ group_offsets, int n_lists, int64_t n_groups, int code_bytes, int chunk_width, int pq_dim, int bits,
                  int in_lds, uint32_t* __restrict__ radii2) {
    extern __shared__ float s_norms[];
    const int n_words = pq_dim << bits;
    if (in_lds)
        for (int i = threadIdx.x; i < n_words; i += blockDim.x) s_norms[i] = word_norms[i];
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), per_word = chunk_width / 4;
    const int64_t n_waves = (int64_t)gridDim.x * (blockDim.x >> 6), wave = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int64_t g0 = n_groups * wave / n_waves, g1 = n_groups * (wave + 1) / n_waves;
    int lo = 0, hi = n_lists;                          // the last list that starts at or before group g0
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (group_offsets[mid] <= g0) lo = mid; else hi = mid;
    }
    const uint32_t mask = (1u << bits) - 1u;
    float mx = 0.f;
    auto give = [&]() {
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
        if (lane == 0 && mx > 0.f) atomicMax(&radii2[lo], __float_as_uint(mx));
        mx = 0.f;
    };
    for (int64_t g = g0; g < g1; ++g) {
        if (group_offsets[lo + 1] <= g) {
            give();
            while (group_offsets[lo + 1] <= g) ++lo;
        }
        const uint32_t* w = reinterpret_cast<const uint32_t*>(codes + g * 64 * code_bytes);
        auto word = [&](int i) { return w[((i / per_word) * 64 + lane) * per_word + i % per_word]; };
        float sum = 0.f;
        uint64_t held = 0;
        int have = 0, next = 0;
        for (int j = 0; j < pq_dim; ++j) {
            if (have < bits) { held |= (uint64_t)word(next++) << have; have += 32; }
            const uint32_t at = ((uint32_t)j << bits) + ((uint32_t)held & mask);
            sum += in_lds ? s_norms[at] : word_norms[at];
            held >>= bits;
            have -= bits;
        }
        if (list_offsets[lo] + (g - group_offsets[lo]) * 64 + lane < list_offsets[lo + 1]) mx = fmaxf(mx, sum);
    }
    if (g0 < g1) give();
}

int upload_impl(ivfpq_index_t* idx, void* d_buf, size_t bytes, void* hip_stream) {
    if (!idx || !d_buf) return fail(IVFPQ_EINVAL, "ivfpq_upload: null pointer");
    const ImageLayout L = image_layout(idx);
    if (bytes < L.total) return fail(IVFPQ_ENOSPACE, "device buffer of %zu bytes given, %zu needed", bytes, L.total);
    if (((uintptr_t)d_buf % kAlign) != 0) return fail(IVFPQ_EINVAL, "device buffer must be %zu-byte aligned", kAlign);
    if (idx->total_groups >= ((int64_t)1 << 32))
        return fail(IVFPQ_EUNSUPPORTED, "%lld 64-vector groups (limit 2^32)", (long long)idx->total_groups);
    hipStream_t st = (hipStream_t)hip_stream;
    unsigned char* base = (unsigned char*)d_buf;
    const int cb = idx->code_bytes(), cw = chunk_width(idx), nch = cb / cw;
    // Everything before the codes is put together on the host and travels as one (a copy of a few kB costs what 1 MB costs), behind the
    // first codes.  The norms in it and the sample that filter_pays needs are made beside the transfers, which one thread of the host stages.
    const size_t n_words = (size_t)idx->pq_dim << idx->pq_bits;
    ivfpq::HostArray<unsigned char> head(L.codes);
    float cn_max = 0.f, wn_max = 0.f;
    bool moderate = true;
    auto norms = [&] {
        float* cnorm = (float*)(head.data() + L.centroid_norms);
        for (int l = 0; l < idx->n_lists; l += 8) {                                       // eight sums at a time: each is one chain of additions
            double acc[8] = {};
            const float* c[8];
            for (int u = 0; u < 8; ++u) c[u] = idx->centroids.data() + (size_t)std::min(l + u, idx->n_lists - 1) * idx->d;
            for (int t = 0; t < idx->d; ++t)
                for (int u = 0; u < 8; ++u) { double v = c[u][t]; acc[u] += v * v; }
            for (int u = 0; u < 8 && l + u < idx->n_lists; ++u) {
                cnorm[l + u] = (float)acc[u];
                if (cnorm[l + u] > cn_max) cn_max = cnorm[l + u];
            }
        }
        float* wnorm = (float*)(head.data() + L.word_norms);
        for (size_t i = 0; i < n_words; ++i) {
            float acc = 0.f;
            for (int t = 0, m = idx->m(); t < m; ++t) { const float v = idx->codebooks[i * m + t]; acc += v * v; }
            wnorm[i] = acc;
            moderate = moderate && acc <= 1e28f;
            wn_max = std::max(wn_max, acc);
        }
    };
    ivfpq::PassShares shares;
    const bool may_filter = filter_supported(idx->pq_bits, idx->pq_dim, idx->d, cw);
    std::memset(head.data(), 0, head.size());
    std::atomic<bool> normed{false};
    ivfpq::SideTask aside([&] {
        norms();
        normed.store(true, std::memory_order_release);
        if (may_filter) shares = ivfpq::sample_pass_shares(*idx);
    });
    std::memcpy(head.data() + L.centroids, idx->centroids.data(), idx->centroids.size() * 4);
    std::memcpy(head.data() + L.codebooks, idx->codebooks.data(), idx->codebooks.size() * 4);
    std::memcpy(head.data() + L.list_offsets, idx->list_offsets.data(), idx->list_offsets.size() * 8);
    uint32_t* sizes = (uint32_t*)(head.data() + L.list_sizes);
    int64_t* goff = (int64_t*)(head.data() + L.group_offsets);
    for (int l = 0; l < idx->n_lists; ++l) {
        int64_t len = idx->list_offsets[l + 1] - idx->list_offsets[l];
        sizes[l] = (uint32_t)len;
        goff[l + 1] = goff[l] + (len + 63) / 64;
    }
    bool head_sent = false;
    auto send_head = [&]() -> int {
        if (head_sent) return IVFPQ_OK;
        while (!normed.load(std::memory_order_acquire)) std::this_thread::yield();
        HIP_TRY(hipMemcpyAsync(base, head.data(), head.size(), hipMemcpyHostToDevice, st));
        head_sent = true;
        return IVFPQ_OK;
    };
    // The codes travel in list order, as many whole groups at a time as fit the place of the ids, and are interleaved
    // from there on the device; the ids follow.
    const int64_t cap = idx->n == 0 ? 0 : (int64_t)((L.total - L.ids) / (size_t)cb);      // vectors in transit, 64 or more
    int64_t g = 0, v = 0;
    while (v < idx->n) {
        int64_t g_end = idx->total_groups, v_end = idx->n;
        if (idx->n - v > cap) {
            const int l = (int)(std::upper_bound(idx->list_offsets.begin(), idx->list_offsets.end(), v + cap) - idx->list_offsets.begin()) - 1;
            const int64_t whole = (v + cap - idx->list_offsets[l]) / 64;
            g_end = goff[l] + whole;
            v_end = idx->list_offsets[l] + whole * 64;
        }
        const size_t blocks = (size_t)(g_end - g + 3) / 4;
        if (g_end <= g || v_end - v > cap || blocks > 0x7FFFFFFFull)
            return fail(IVFPQ_EUNSUPPORTED, "internal: %lld code groups in transit", (long long)(g_end - g));
        HIP_TRY(hipMemcpyAsync(base + L.ids, idx->codes.data() + (size_t)v * cb, (size_t)(v_end - v) * cb, hipMemcpyHostToDevice, st));
        if (int s = send_head()) return s;
        auto launch = [&](auto zero) {
            using W = decltype(zero);
            hipLaunchKernelGGL(interleave_codes_kernel<W>, dim3((unsigned)blocks), dim3(256), 0, st, (const W*)(base + L.ids), v,
                               (const int64_t*)(base + L.list_offsets), (const int64_t*)(base + L.group_offsets), idx->n_lists, g, g_end,
                               nch, (W*)(base + L.codes));
        };
        if (cw == 16) launch(uint4{}); else launch(uint32_t{});
        HIP_TRY(hipGetLastError());
        g = g_end;
        v = v_end;
    }
    if (int s = send_head()) return s;
    if (idx->total_groups > 0) {
        const bool in_lds = n_words * 4 <= kLdsBytes;
        if (int s = allow_full_lds(list_radii_kernel)) return s;
        const unsigned radii_blocks = (unsigned)std::min<int64_t>(512, (idx->total_groups + 15) / 16);
        hipLaunchKernelGGL(list_radii_kernel, dim3(radii_blocks), dim3(1024), in_lds ? n_words * 4 : 0, st, (const unsigned char*)(base + L.codes),
                           (const float*)(base + L.word_norms), (const int64_t*)(base + L.list_offsets), (const int64_t*)(base + L.group_offsets),
                           idx->n_lists, idx->total_groups, cb, cw, idx->pq_dim, idx->pq_bits, in_lds, (uint32_t*)(base + L.list_radii));
        HIP_TRY(hipGetLastError());
    }
    if (idx->n > 0)
        HIP_TRY(hipMemcpyAsync(base + L.ids, idx->ids.data(), idx->ids.size() * 8, hipMemcpyHostToDevice, st));
    const ivfpq::RankCrowd crowd = ivfpq::sample_rank_crowd(*idx, cn_max);          // (while the last kernels run; the head had the norms)
    HIP_TRY(hipStreamSynchronize(st));
    aside.wait();
    idx->pass_shares = shares;
    idx->rank_crowd = crowd;
    idx->centroid_norm_max = cn_max;
    idx->word_norm_max = moderate ? std::sqrt(wn_max) * kWordNormSlack : -1.f;

    // set-up of the static scratch for this device (ivfpq_search_static looks it up here, not in the hot loop)
    void* scratch_dev = nullptr;
    if (int s = static_scratch_ptr(&scratch_dev)) return s;
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    idx->dev.valid = true;
    idx->dev.device = dev;
    idx->dev.centroids = (const float*)(base + L.centroids);
    idx->dev.centroid_norms = (const float*)(base + L.centroid_norms);
    idx->dev.codebooks = (const float*)(base + L.codebooks);
    idx->dev.list_offsets = (const int64_t*)(base + L.list_offsets);
    idx->dev.list_sizes = (const uint32_t*)(base + L.list_sizes);
    idx->dev.list_radii = (const float*)(base + L.list_radii);
    idx->dev.group_offsets = (const int64_t*)(base + L.group_offsets);
    idx->dev.codes = (const uint8_t*)(base + L.codes);
    idx->dev.ids = (const int64_t*)(base + L.ids);
    return IVFPQ_OK;
}
}  // namespace

extern "C" {

int ivfpq_upload(ivfpq_index_t* idx, void* d_buf, size_t bytes, void* hip_stream) {
    return guarded("ivfpq_upload", [&] { return upload_impl(idx, d_buf, bytes, hip_stream); });
}

size_t ivfpq_search_workspace_bytes(const ivfpq_index_t* index, int64_t nq, int32_t n_probes, int32_t k,
                                    int32_t lut_dtype) {
    (void)k; (void)lut_dtype;
    if (!index || n_probes < 1 || nq < 0) { set_error("ivfpq_search_workspace_bytes: bad arguments"); return 0; }
    Plan own, given;   // large enough for ivfpq_search and for ivfpq_search_with_probes
    if (make_plan(index, nq, n_probes, false, &own) != IVFPQ_OK) return 0;
    if (make_plan(index, nq, n_probes, true, &given) != IVFPQ_OK) return 0;
    return std::max(own.total, given.total);
}

int ivfpq_search(const ivfpq_index_t* index, const float* d_queries, int64_t nq, int32_t n_probes, int32_t k,
                 int32_t lut_dtype, int64_t* d_ids, float* d_dists, void* d_workspace, size_t workspace_bytes,
                 void* hip_stream) {
    return guarded("ivfpq_search", [&] {
        return search_impl(index, d_queries, nq, nullptr, n_probes, k, lut_dtype, d_ids, d_dists, d_workspace,
                           workspace_bytes, hip_stream);
    });
}

int ivfpq_search_static(const ivfpq_index_t* index, const float* d_queries, int64_t nq, int32_t n_probes, int32_t k,
                        int32_t lut_dtype, int64_t* d_ids, float* d_dists, void* hip_stream) {
    return guarded("ivfpq_search_static", [&] {
        return search_impl(index, d_queries, nq, nullptr, n_probes, k, lut_dtype, d_ids, d_dists, nullptr, 0,
                           hip_stream, true);
    });
}

int ivfpq_search_with_probes(const ivfpq_index_t* index, const float* d_queries, int64_t nq,
                             const uint32_t* d_probes, int32_t n_probes, int32_t k, int32_t lut_dtype,
                             int64_t* d_ids, float* d_dists, void* d_workspace, size_t workspace_bytes,
                             void* hip_stream) {
    if (nq > 0 && !d_probes) return fail(IVFPQ_EINVAL, "ivfpq_search_with_probes: null probes");
    return guarded("ivfpq_search_with_probes", [&] {
        return search_impl(index, d_queries, nq, d_probes, n_probes, k, lut_dtype, d_ids, d_dists, d_workspace,
                           workspace_bytes, hip_stream);
    });
}

int ivfpq_select_probes(const ivfpq_index_t* idx, const float* d_queries, int64_t nq, int32_t n_probes,
                        uint32_t* d_probes, float* d_probe_dists, void* d_workspace, size_t workspace_bytes,
                        void* hip_stream) {
    if (int s = check_search_args(idx, d_queries, nq, n_probes, 1, 0, false)) return s;
    if (nq > 0 && !d_probes) return fail(IVFPQ_EINVAL, "ivfpq_select_probes: null output");
    if (int s = check_device(idx)) return s;
    if (nq == 0) return IVFPQ_OK;
    Plan plan;
    if (int s = make_plan(idx, nq, n_probes, false, &plan)) return s;
    if (!d_workspace || workspace_bytes < plan.total)
        return fail(IVFPQ_ENOSPACE, "workspace of %zu bytes given, %zu needed", workspace_bytes, plan.total);
    hipStream_t st = (hipStream_t)hip_stream;
    float* w_D = (float*)((unsigned char*)d_workspace + plan.D);
    StripSummary* w_S = (StripSummary*)((unsigned char*)d_workspace + plan.S);
    for (int64_t q0 = 0; q0 < nq; q0 += plan.tile) {
        const int tq = (int)std::min<int64_t>(plan.tile, nq - q0);
        StripSummary* strips = w_S;
        bool exact = false;
        if (int s = launch_step_1a(idx, d_queries + (size_t)q0 * idx->d, tq, n_probes, (uint32_t*)w_D, &strips, &exact,
                                   (unsigned char*)d_workspace + plan.split, st))
            return s;
        launch_select_probes((int)tq, exact, st, (uint32_t*)w_D, (const StripSummary*)strips,
                             coarse_strip_width(tq, idx->n_lists), d_queries + (size_t)q0 * idx->d, idx->dev.centroids, idx->centroid_norm_max, idx->rank_crowd, idx->d,
                             idx->n_lists, n_probes, idx->dev.list_sizes, idx->dev.group_offsets, d_probes + (size_t)q0 * n_probes,
                             d_probe_dists ? d_probe_dists + (size_t)q0 * n_probes : nullptr, (uint32_t*)nullptr,
                             (uint4*)nullptr, 0);
        HIP_TRY(hipGetLastError());
    }
    return IVFPQ_OK;
}

int ivfpq_dump_lut(const ivfpq_index_t* idx, const float* d_query, uint32_t list_id, int32_t lut_dtype,
                   void* d_lut_out, void* hip_stream) {
    if (!idx || !d_query || !d_lut_out) return fail(IVFPQ_EINVAL, "ivfpq_dump_lut: null pointer");
    if (lut_dtype < 0 || lut_dtype > 3) return fail(IVFPQ_EINVAL, "unknown lut_dtype %d", lut_dtype);
    if (list_id >= (uint32_t)idx->n_lists) return fail(IVFPQ_EINVAL, "list_id %u >= n_lists %d", list_id, idx->n_lists);
    if (int s = check_device(idx)) return s;
    const size_t lds = scan_lds_bytes(idx, lut_dtype);
    if (lds > kLdsBytes) return fail(IVFPQ_EUNSUPPORTED, "lookup table needs %zu bytes of LDS (limit %zu)", lds, kLdsBytes);
    hipStream_t st = (hipStream_t)hip_stream;
    const float* centroid = idx->dev.centroids + (size_t)list_id * idx->d;
    auto go = [&](auto kernel) -> int {
        if (int s = allow_full_lds(kernel)) return s;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(256), lds, st, d_query, centroid, idx->dev.codebooks, idx->d,
                           idx->pq_dim, idx->m(), idx->pq_bits, fp8_mode(idx, lut_dtype), (unsigned char*)d_lut_out);
        HIP_TRY(hipGetLastError());
        return IVFPQ_OK;
    };
    switch (lut_dtype) {
        case IVFPQ_LUT_FP32: return go(dump_lut_kernel<IVFPQ_LUT_FP32>);
        case IVFPQ_LUT_FP16: return go(dump_lut_kernel<IVFPQ_LUT_FP16>);
        case IVFPQ_LUT_FP8_E5M3: return go(dump_lut_kernel<IVFPQ_LUT_FP8_E5M3>);
        default: return go(dump_lut_kernel<IVFPQ_LUT_FP8_E4M4>);
    }
}

int ivfpq_scan_list(const ivfpq_index_t* idx, const float* d_query, uint32_t list_id, int32_t lut_dtype,
                    float* d_R_out, void* hip_stream) {
    if (!idx || !d_query) return fail(IVFPQ_EINVAL, "ivfpq_scan_list: null pointer");
    if (lut_dtype < 0 || lut_dtype > 3) return fail(IVFPQ_EINVAL, "unknown lut_dtype %d", lut_dtype);
    if (list_id >= (uint32_t)idx->n_lists) return fail(IVFPQ_EINVAL, "list_id %u >= n_lists %d", list_id, idx->n_lists);
    if (int s = check_device(idx)) return s;
    if (idx->list_offsets[list_id + 1] == idx->list_offsets[list_id]) return IVFPQ_OK;
    if (!d_R_out) return fail(IVFPQ_EINVAL, "ivfpq_scan_list: null output");
    ScanArgs a = base_scan_args(idx, lut_dtype);
    a.queries = d_query; a.R = d_R_out; a.single_list = (int)list_id; a.n_probes = 1;
    return launch_scan(idx, a, lut_dtype, dim3(1), (hipStream_t)hip_stream);
}

int ivfpq_refine(const float* d_data, int64_t n_data, int32_t d, const float* d_queries, int64_t nq,
                 const int64_t* d_cand_ids, int32_t n_cand, int32_t k, int64_t* d_ids, float* d_dists, void* hip_stream) {
    if (nq < 0 || n_data < 0 || d < 1) return fail(IVFPQ_EINVAL, "ivfpq_refine: bad shape");
    if (n_cand < 1 || n_cand > IVFPQ_MAX_K) return fail(IVFPQ_EINVAL, "n_cand=%d outside [1, %d]", n_cand, IVFPQ_MAX_K);
    if (k < 1 || k > IVFPQ_MAX_K) return fail(IVFPQ_EINVAL, "k=%d outside [1, %d]", k, IVFPQ_MAX_K);
    if (nq == 0) return IVFPQ_OK;
    if (!d_queries || !d_cand_ids || !d_ids || !d_dists || (n_data > 0 && !d_data))
        return fail(IVFPQ_EINVAL, "ivfpq_refine: null pointer");
    if (nq > 0x7FFFFFFF) return fail(IVFPQ_EUNSUPPORTED, "ivfpq_refine: nq=%lld (limit 2^31 - 1 per call)", (long long)nq);
    hipLaunchKernelGGL(refine_kernel, dim3((unsigned)nq), dim3(SEL_THREADS), 0, (hipStream_t)hip_stream, d_data,
                       (long long)n_data, d, d_queries, d_cand_ids, n_cand, k, d_ids, d_dists);
    HIP_TRY(hipGetLastError());
    return IVFPQ_OK;
}

int ivfpq_stream_read(const void* d_buf, size_t bytes, uint32_t* d_out, int32_t n_out, void* hip_stream) {
    if (!d_buf || !d_out) return fail(IVFPQ_EINVAL, "null pointer");
    if (n_out < 1 || n_out > 65536) return fail(IVFPQ_EINVAL, "n_out=%d outside 1..65536", n_out);
    if (((uintptr_t)d_buf & 15) != 0 || (bytes & 15) != 0) return fail(IVFPQ_EINVAL, "buffer and size must be multiples of 16 bytes");
    hipLaunchKernelGGL(stream_read_kernel, dim3(n_out), dim3(256), 0, (hipStream_t)hip_stream,
                       (const uint4*)d_buf, bytes / 16, d_out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(IVFPQ_EHIP, "stream_read_kernel launch failed: %s", hipGetErrorString(e));
    return IVFPQ_OK;
}

int ivfpq_scan_kernel_info(const ivfpq_index_t* idx, int32_t lut_dtype, char* buf, size_t buf_bytes) {
    if (!idx || !buf || buf_bytes == 0) return fail(IVFPQ_EINVAL, "ivfpq_scan_kernel_info: null pointer");
    if (lut_dtype < 0 || lut_dtype > 3) return fail(IVFPQ_EINVAL, "unknown lut_dtype %d", lut_dtype);
    if (idx->timing && idx->scan_kernel_lut == lut_dtype) {
        snprintf(buf, buf_bytes, "%s", idx->scan_kernel);
        return IVFPQ_OK;
    }
    const uint32_t blk = idx->tuning.order_block > 0 ? (uint32_t)idx->tuning.order_block : kOrderBlock;
    const Fp8Mode fp8 = fp8_mode(idx, lut_dtype);
    const bool grouped = idx->tuning.scan_route == 0 || idx->tuning.scan_route == (int)ScanRoute::kGrouped;      // 0: what large batches take
    const int G = grouped ? scan_group_width(idx, lut_dtype, fp8, blk) : 0;
    if (grouped && filter_applies(idx, lut_dtype, fp8)) describe_filter(idx, lut_dtype, buf, buf_bytes);
    else if (G) describe_group(idx, lut_dtype, G, buf, buf_bytes);
    else describe_scan(idx, lut_dtype, scan_threads(idx, lut_dtype), buf, buf_bytes);
    return IVFPQ_OK;
}

int ivfpq_set_stage_timing(ivfpq_index_t* index, int32_t enabled) {
    if (!index) return fail(IVFPQ_EINVAL, "null index");
    index->timing = enabled != 0;
    index->stage_valid = false;
    index->scan_kernel_lut = -1;
    return IVFPQ_OK;
}

int ivfpq_stage_times_ms(ivfpq_index_t* index, float ms[8]) {
    if (!index || !ms) return fail(IVFPQ_EINVAL, "null pointer");
    if (!index->timing || !index->stage_valid) return fail(IVFPQ_ESTATE, "no timed search call recorded");
    for (int i = 0; i < 8; ++i) ms[i] = 0.f;
    for (const auto& sp : index->spans) {
        float t = 0.f;
        HIP_TRY(hipEventElapsedTime(&t, (hipEvent_t)sp.a, (hipEvent_t)sp.b));
        ms[sp.stage] += t * sp.share;
    }
    return IVFPQ_OK;
}

}  // extern "C"
