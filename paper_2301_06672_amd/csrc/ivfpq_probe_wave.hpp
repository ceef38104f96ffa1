// Step 1b for large batches: the n_probes <= 64 nearest clusters of a query by one wave.  Included by ivfpq_device.hip only; the code has
// internal linkage.
#pragma once

#include <hip/hip_runtime.h>

#include "ivfpq_lds_util.hpp"
#include "ivfpq_rank.hpp"
#include "ivfpq_select.hpp"

namespace {

// As select_probes_kernel, which takes a workgroup and some twenty barriers a query: candidates by ranking value within its error bound, exact
// distances for them, the n_probes nearest of those in order, the query's descriptors.  Here
//   - the bound on the n_probes-th smallest ranking value is that of 256 minima (four to a lane, of interleaved shares of the row), by
//     bisection over their bits with ballots;
//   - candidates are ranked by counting, 192 at a time: where more are within the error bound (it goes with the norms; an index whose vectors
//     share an offset has hundreds, and is left to workgroups, but a query may lie far out) the nearest so far stay and the next join them.  8,000 clusters of 128 components, 64 probes, 4,096
//     queries, ranking included: centred 119 us by workgroups and 108 by waves, offset by 400 167 and 164 (4,023 with all clusters' distances and a
//     pass over them a probe); 2,000 clusters, 10,000 queries 168 and 154 (812).
// Bound by the instructions and the waits of one wave, of which the chip holds 8,192 at once: 10,000 queries on 1,024 clusters, 20 probes,
// 66 -> 29 us; 2,000, 64 probes, 108 -> 61; 4,096 queries on 1,024 30 -> 15.  (Strip summaries yield five times as many candidates, whose
// distances are too much for one wave: 10,000 clusters, 50 probes, 95 us by workgroups, 173 by waves.)
using ivfpq::kWaveProbes;
using ivfpq::select_by_waves;
constexpr int kWaveCand = 192, kWaveQueries = 4;
static_assert(kWaveProbes + kWave <= kWaveCand, "the nearest so far leave room for a step of the row");

__global__ void __launch_bounds__(64 * kWaveQueries)
select_probes_wave_kernel(uint32_t* __restrict__ A, const float* __restrict__ queries, const float* __restrict__ centroids, float centroid_norm_max, int d, int n_lists, int n_probes, int nq,
                          const uint32_t* __restrict__ list_sizes, const int64_t* __restrict__ group_offsets,
                          uint32_t* __restrict__ probes, float* __restrict__ probe_dists, uint32_t* __restrict__ roff, uint4* __restrict__ pairs, int k_hint,
                          uint32_t* __restrict__ nearest) {
    constexpr int kHeld = kWaveCand / kWave;
    __shared__ unsigned long long s_key[kWaveQueries][kWaveCand];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t q = blockIdx.x * (uint32_t)kWaveQueries + (uint32_t)wave;
    if (q >= (uint32_t)nq) return;
    const float* const qv = queries + (size_t)q * d;
    uint32_t* const row = A + (size_t)q * n_lists;
    unsigned long long* const keys = s_key[wave];                     // cluster; distance (high half) and cluster, once that is known
    auto settle = [&]() __attribute__((always_inline)) {               // the wave's own LDS writes are in place
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    // sink(key, index, share 0 ... 3) of every ranking value; whole waves, invalid ones with the index -1.  more(n): the first n are done
    const uint32_t n_keys = (uint32_t)n_lists;
    auto each_key = [&](auto sink, auto more) __attribute__((always_inline)) {
        if ((n_lists & 3) == 0) {
            const uint4* const row4 = reinterpret_cast<const uint4*>(row);
#pragma unroll 1
            for (uint32_t base = 0; base < n_keys / 4u; base += 4u * kWave) {
                uint4 v[4];
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    const uint32_t i = base + u * kWave + (uint32_t)lane;
                    v[u] = row4[i < n_keys / 4u ? i : 0u];
                }
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    const uint32_t i = base + u * kWave + (uint32_t)lane;
                    const bool in = i < n_keys / 4u;
                    sink(v[u].x, in ? (int)(4u * i) : -1, 0); sink(v[u].y, in ? (int)(4u * i + 1u) : -1, 1);
                    sink(v[u].z, in ? (int)(4u * i + 2u) : -1, 2); sink(v[u].w, in ? (int)(4u * i + 3u) : -1, 3);
                }
                if (!more(4u * base + 16u * kWave)) return;
            }
        } else {
#pragma unroll 1
            for (uint32_t base = 0; base < n_keys; base += 4u * kWave) {
                uint32_t v[4];
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    const uint32_t i = base + u * kWave + (uint32_t)lane;
                    v[u] = row[i < n_keys ? i : 0u];
                }
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    const uint32_t i = base + u * kWave + (uint32_t)lane;
                    sink(v[u], i < n_keys ? (int)i : -1, (int)u);
                }
                if (!more(base + 4u * kWave)) return;
            }
        }
    };
    uint32_t least[4] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
    each_key([&](uint32_t key, int i, int share) __attribute__((always_inline)) { least[share] = i >= 0 && key < least[share] ? key : least[share]; },
             [](uint32_t) { return true; });
    // |q|^2, for the error bound of the ranking values
    float qn = 0.f;
    for (int c = lane; c < d; c += kWave) qn = __builtin_fmaf(qv[c], qv[c], qn);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) qn += __shfl_xor(qn, off, kWave);
    // n_probes of the minima are not above this (bits from the 9th on), and with them as many ranking values
    uint32_t kth = 0;
#pragma unroll 1
    for (int bit = 31; bit >= 8; --bit) {                             // the largest number with fewer than n_probes minima below it
        const uint32_t tried = kth | 1u << bit;
        uint32_t less = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) less += (uint32_t)__popcll(ballot64(least[u] < tried));
        if (less < (uint32_t)n_probes) kth = tried;
    }
    uint32_t limit;
    {
        const float f = ordered_key_value(kth | 0xFFu);
        float g = f + 2.f * rank_error_bound(d, qn, centroid_norm_max);
        g += __builtin_fabsf(g) * 2.3841858e-07f;                     // the addition above rounds: stay on the safe side
        limit = g == g ? ordered_key(g) : 0xFFFFFFFFu;                // NaN (from infinite inputs): admit everything
    }
    uint32_t n = 0;                                                   // candidates in keys; the same for the whole wave
    auto append = [&](bool has, uint32_t cluster) __attribute__((always_inline)) {
        const unsigned long long m = ballot64(has);
        const uint32_t slot = n + lanes_below(m);
        if (has && slot < (uint32_t)kWaveCand) keys[slot] = cluster;
        n += (uint32_t)__popcll(m);
    };
    // More than the buffer holds (vectors that share an offset: the error bound grows with the norms): from the last step after which it held
    // them on, the row is taken as many candidates at a time as fit beside the nearest so far.
    uint32_t at = n_keys, n_held = 0, at_held = 0;                    // the row from `at` on is not in the buffer yet
    each_key([&](uint32_t key, int i, int) __attribute__((always_inline)) {
        const bool in = i >= 0 && key <= limit;
        if (ballot64(in) != 0) append(in, (uint32_t)i);
    }, [&](uint32_t done) {
        if (n > (uint32_t)kWaveCand) return false;
        n_held = n;
        at_held = done;
        return true;
    });
    if (n > (uint32_t)kWaveCand) { n = n_held; at = at_held; }
    else if (n < (uint32_t)n_probes) { n = 0; at = 0; limit = 0xFFFFFFFFu; }        // not-a-number keys are above every limit: all clusters
    // exact squared distances in direct form: the sum of select_probes_kernel, a group of 8 adjacent lanes per cluster, two clusters a group
    // under way together
    auto distances = [&](uint32_t n, auto cluster_of, auto sink) __attribute__((always_inline)) {
#pragma unroll 1
        for (uint32_t base = 0; base < n; base += 16) {
            const uint32_t j0 = base + (uint32_t)(lane >> 3), j1 = j0 + 8u;
            const bool v0 = j0 < n, v1 = j1 < n;
            const float *c0 = centroids + (size_t)(v0 ? cluster_of(j0) : 0u) * d, *c1 = centroids + (size_t)(v1 ? cluster_of(j1) : 0u) * d;
            float a0 = 0.f, a1 = 0.f;
#pragma unroll 8
            for (int u = lane & 7; u < d; u += 8) {
                const float x = qv[u], d0 = x - c0[u], d1 = x - c1[u];
                a0 = __builtin_fmaf(d0, d0, a0);
                a1 = __builtin_fmaf(d1, d1, a1);
            }
            a0 = sum_over_8_lanes(a0);
            a1 = sum_over_8_lanes(a1);
            if ((lane & 7) == 0) {
                if (v0) sink(j0, a0);
                if (v1) sink(j1, a1);
            }
        }
    };
    auto key_of = [](float dist, uint32_t cluster) { return (unsigned long long)__float_as_uint(dist) << 32 | cluster; };
    uint32_t n_kept = 0;                                              // keys[0 .. n_kept): the nearest so far, in order
    for (;;) {
        if (at < n_keys) {
            auto key_at = [&](uint32_t i) { return row[i < n_keys ? i : 0u]; };
            uint32_t ahead = key_at(at + (uint32_t)lane);
#pragma unroll 1
            for (; at < n_keys && n + (uint32_t)kWave <= (uint32_t)kWaveCand; at += kWave) {
                const uint32_t i = at + (uint32_t)lane, key = ahead;
                ahead = key_at(i + kWave);
                append(key <= limit && i < n_keys, i);
            }
        }
        settle();
        const uint32_t first = n_kept;
        distances(n - first, [&](uint32_t j) { return (uint32_t)keys[first + j]; },
                  [&](uint32_t j, float dist) { keys[first + j] = key_of(dist, (uint32_t)keys[first + j]); });
        settle();
        unsigned long long key[kHeld];
#pragma unroll
        for (int u = 0; u < kHeld; ++u) key[u] = (uint32_t)(u * kWave + lane) < n ? keys[u * kWave + lane] : ~0ull;
        if (first == (uint32_t)n_probes) {                            // what is nearer than the last of these, moved up to them
            const unsigned long long last = keys[first - 1u];
            settle();
            n = first;
#pragma unroll
            for (int u = 0; u < kHeld; ++u) {
                const bool in = (uint32_t)(u * kWave + lane) >= first && key[u] < last;
                const unsigned long long m = ballot64(in);
                if (in) keys[n + lanes_below(m)] = key[u];
                n += (uint32_t)__popcll(m);
            }
            settle();
#pragma unroll
            for (int u = 0; u < kHeld; ++u) key[u] = (uint32_t)(u * kWave + lane) < n ? keys[u * kWave + lane] : ~0ull;
        }
        uint32_t rank[kHeld] = {};
#pragma unroll 1
        for (uint32_t j = 0; n != first && j < n; j += 2) {
            const unsigned long long k0 = keys[j], k1 = j + 1u < n ? keys[j + 1u] : ~0ull;
#pragma unroll
            for (int u = 0; u < kHeld; ++u)
                if ((uint32_t)(u * kWave) < n) rank[u] += (k0 < key[u] ? 1u : 0u) + (k1 < key[u] ? 1u : 0u);
        }
        settle();
#pragma unroll
        for (int u = 0; u < kHeld; ++u)
            if (n != first && (uint32_t)(u * kWave + lane) < n && rank[u] < (uint32_t)n_probes) keys[rank[u]] = key[u];
        settle();
        n_kept = n < (uint32_t)n_probes ? n : (uint32_t)n_probes;
        if (at >= n_keys) break;
        n = n_kept;
    }
    const unsigned long long mine = lane < n_probes ? keys[lane] : ~0ull;      // of lane p < n_probes: the p-th nearest, distance and cluster
    uint32_t l = lane < n_probes ? (uint32_t)mine : 0u;
    float dist = __uint_as_float((uint32_t)(mine >> 32));
    if (!roff) {                                                      // the caller's probe lists: nearest first
        if (lane < n_probes) {
            probes[(size_t)q * n_probes + lane] = l;
            if (probe_dists) probe_dists[(size_t)q * n_probes + lane] = dist;
        }
        return;
    }
    // The search's own lists, as in select_probes_kernel: slot 0 is the nearest cluster that holds at least k_hint vectors.
    uint32_t len = lane < n_probes ? list_sizes[l] : 0u, group = lane < n_probes ? (uint32_t)group_offsets[l] : 0u;
    const unsigned long long large = k_hint > 0 ? ballot64(lane < n_probes && len >= (uint32_t)k_hint) : 0ull;
    const int pivot = large != 0 ? __ffsll((long long)large) - 1 : 0, from = lane == 0 ? pivot : lane <= pivot ? lane - 1 : lane;
    l = (uint32_t)__shfl((int)l, from, kWave);
    len = (uint32_t)__shfl((int)len, from, kWave);
    group = (uint32_t)__shfl((int)group, from, kWave);
    dist = __shfl(dist, from, kWave);
    const uint32_t padded = lane < n_probes ? (len + 63u) & ~63u : 0u, upto = wave_inclusive_scan(padded);
    if (lane < n_probes) {
        probes[(size_t)q * n_probes + lane] = l;
        if (probe_dists) probe_dists[(size_t)q * n_probes + lane] = dist;
        roff[(size_t)q * (n_probes + 1) + lane] = upto - padded;
        pairs[(size_t)q * n_probes + lane] = make_uint4(l, len, group, upto - padded);
    }
    if (nearest && lane == 0) nearest[q] = l;
    if (lane == kWave - 1) roff[(size_t)q * (n_probes + 1) + n_probes] = upto;
}

}  // namespace
