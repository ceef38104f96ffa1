// The bound of a query from the values of its nearest probe, by one wave.  Included by ivfpq_device.hip only; the code has internal linkage.
#pragma once

#include <hip/hip_runtime.h>

#include "ivfpq_lds_util.hpp"
#include "ivfpq_nearest_rules.hpp"
#include "ivfpq_scan_args.hpp"
#include "ivfpq_select.hpp"

namespace {

// What bound_of_nearest does at the end of a workgroup that has scanned its query's nearest probe, for probes scanned by the group kernel, whose
// workgroups have several queries: the k-th smallest of row[0 .. len) bounds the query's k-th smallest R; it and what is not above it
// become the first entries of the survivor list.  Fewer than k finite values: no bound, every vector is admitted.
// The k-th smallest of 256 minima (four to a lane, of interleaved shares of the list) is not below the k-th smallest value: what is not above
// it is gathered and the k-th found exactly, by bisection over the bits with ballots.  More than a wave has room for (rare up to k = 100, one
// query in 25 at 128; values that cluster): the bound is that minimum, and a few values too many are listed; the selection at the end is exact.
using ivfpq::kBoundCand;
using ivfpq::kBoundWaveK;
constexpr int kBoundQueries = 4;
static_assert(ivfpq::kBoundShares == 4 * kWave && kBoundCand % kWave == 0, "four minima a lane, whole registers of values");

__global__ void __launch_bounds__(64 * kBoundQueries)
bound_wave_kernel(ivfpq::ScanArgs a, int nq) {
    __shared__ uint2 s_cand[kBoundQueries][kBoundCand];
#pragma unroll
    for (int c = 0; c < 2; ++c)                                       // the counters of the grouping that follows
        for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < a.n_clear[c]; i += gridDim.x * blockDim.x) a.clear[c][i] = 0u;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t q = blockIdx.x * (uint32_t)kBoundQueries + (uint32_t)wave;
    if (q >= (uint32_t)nq) return;
    uint2* const cand = s_cand[wave];
    const uint32_t len = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.pairs[(size_t)q * a.n_probes].y), seg0 = (len + 63u) & ~63u, k = (uint32_t)a.k_bound;
    uint32_t* const row = reinterpret_cast<uint32_t*>(a.R + (size_t)q * a.stride);          // stride: a multiple of 64
    uint32_t* const row_pos = a.Rpos + (size_t)q * a.stride;
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    // value(key, position, share) of every vector of the list, whole waves, kNone past its end; the first 2,048 stay in registers
    constexpr int kHeld = 8;
    const uint32_t n4 = seg0 / 4u;
    const uint4* const row4 = reinterpret_cast<const uint4*>(row);
    auto load = [&](uint32_t base) __attribute__((always_inline)) {
        const uint32_t i = base + (uint32_t)lane;
        uint4 x = row4[i < n4 ? i : 0u];
        if (4u * base + 4u * kWave > len) {
            x.x = 4u * i < len ? x.x : kNone;
            x.y = 4u * i + 1u < len ? x.y : kNone;
            x.z = 4u * i + 2u < len ? x.z : kNone;
            x.w = 4u * i + 3u < len ? x.w : kNone;
        }
        return x;
    };
    uint4 held[kHeld];
#pragma unroll
    for (int u = 0; u < kHeld; ++u) held[u] = (uint32_t)(u * kWave) < n4 ? load((uint32_t)(u * kWave)) : make_uint4(kNone, kNone, kNone, kNone);
    auto each_value = [&](auto value) __attribute__((always_inline)) {
        auto four = [&](const uint4 x, uint32_t base) __attribute__((always_inline)) {
            const uint32_t i = 4u * (base + (uint32_t)lane);
            value(x.x, i, 0); value(x.y, i + 1u, 1); value(x.z, i + 2u, 2); value(x.w, i + 3u, 3);
        };
#pragma unroll
        for (int u = 0; u < kHeld; ++u)
            if ((uint32_t)(u * kWave) < n4) four(held[u], (uint32_t)(u * kWave));
#pragma unroll 1
        for (uint32_t base = kHeld * kWave; base < n4; base += 4 * kWave) {
            uint4 x[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) x[u] = load(base + u * kWave);
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) four(x[u], base + u * kWave);
        }
    };
    uint32_t n_listed = 0;                                            // the same for the whole wave
    auto append = [&](bool in, uint32_t key, uint32_t i) __attribute__((always_inline)) {
        const unsigned long long m = ballot64(in);
        if (m == 0) return;
        if (in) {
            const uint32_t at = seg0 + n_listed + lanes_below(m);
            row[at] = key;
            row_pos[at] = i;
        }
        n_listed += (uint32_t)__popcll(m);
    };
    uint32_t bound = ivfpq::kAdmitAll;
    bool listed = false;
    if (len >= k) {
        uint32_t least[4] = {kNone, kNone, kNone, kNone};
        each_value([&](uint32_t key, uint32_t, int share) __attribute__((always_inline)) { least[share] = key < least[share] ? key : least[share]; });
        uint32_t upto = 0;                                            // (bits from the 10th on; all below are admitted)
#pragma unroll 1
        for (int bit = 31; bit >= 9; --bit) {
            const uint32_t tried = upto | 1u << bit;
            uint32_t less = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) less += (uint32_t)__popcll(ballot64(least[u] < tried));
            if (less < k) upto = tried;
        }
        upto |= 0x1FFu;
        if (upto < 0x7F800000u) {
            uint32_t n = 0;
            each_value([&](uint32_t key, uint32_t i, int) __attribute__((always_inline)) {
                const bool in = key <= upto;
                const unsigned long long m = ballot64(in);
                if (m == 0) return;
                const uint32_t slot = n + lanes_below(m);
                if (in && slot < (uint32_t)kBoundCand) cand[slot] = make_uint2(key, i);
                n += (uint32_t)__popcll(m);
            });
            bound = upto;
            if (n <= (uint32_t)kBoundCand) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                uint2 mine[kBoundCand / kWave];
#pragma unroll
                for (int u = 0; u < kBoundCand / kWave; ++u) mine[u] = (uint32_t)(u * kWave + lane) < n ? cand[u * kWave + lane] : make_uint2(kNone, 0u);
                bound = 0;
#pragma unroll 1
                for (int bit = 30; bit >= 0; --bit) {                 // the largest number with fewer than k values below it: the k-th
                    const uint32_t tried = bound | 1u << bit;
                    uint32_t less = 0;
#pragma unroll
                    for (int u = 0; u < kBoundCand / kWave; ++u) less += (uint32_t)__popcll(ballot64(mine[u].x < tried));
                    if (less < k) bound = tried;
                }
#pragma unroll
                for (int u = 0; u < kBoundCand / kWave; ++u) append(mine[u].x <= bound, mine[u].x, mine[u].y);
                listed = true;
            }
        }
    }
    if (!listed) each_value([&](uint32_t key, uint32_t i, int) __attribute__((always_inline)) { append(i < len && key <= bound, key, i); });
    if (lane == 0) {
        a.bounds[q] = bound;
        a.counts[q] = n_listed;
        if (a.starts) a.starts[q] = n_listed;
    }
}

}  // namespace
