// The nearest of many centres for every row, as decided by float64 distances (ties to the lower index), with one matrix product in
// half precision.  Included by ivfpq_build.hip only; everything has internal linkage.
//
//   centre_mean / centre_stats / centre_halves / row_halves   x' = x - mean and c' = c - mean, the mean of the centres, scaled by a
//                     power of two and rounded to half, in the layout that a wave reads as matrix operands.  Only differences
//                     of distances count, which a common shift leaves alone while the error below falls with the norms
//   near_kernel       v(x, c) = x'.c' - |c'|^2 / 2 of a tile of rows and all centres, the rows' operands in registers, the centres' streamed
//                     from the L2; per row the largest value, its centre and the second largest.  No value is stored
//   near_decide_kernel    |x - c|^2 = |x'|^2 - 2 v: where the second value is further below the first than twice the error of a value, the
//                     first is the nearest.  The other rows are listed
//   near_kernel (emit)    the listed rows again: every centre within that distance of the first
//   near_exact_kernel     float64 distances of those; near_scan_kernel: of all centres, for rows with more of them than a list holds
//
// Error of a value (near_error): half rounds either operand by 2^-11, so r.y is off by 2^-10 |x'||c'|; the sum of d + 1 terms in fp32 in any
// order (4 (d + 10) 2^-24 of the magnitudes, a factor 4 of slack as for the other ranking values), the position in the low four bits of a value
// (2^-19), operands below the half's normal range.
// 500,000 rows of 96 components against 10,000 centres: 1.3 ms; three products of bf16 halves, summaries of every strip of 64 centres
// stored and read back (nearest_strips_kernel), 4.3 ms.
#pragma once

#include <hip/hip_runtime.h>

#include "ivfpq_lds_util.hpp"
#include "ivfpq_rank.hpp"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int kNearList = 15;                  // centres that a listed row can hold
constexpr int kNearThreads = 256;

// What the launches share, on the device: the mean of the centres, the largest |c'| component and |c'|^2 (bit patterns), the number of
// listed rows and of those that scan all centres.
struct NearStats {
    uint32_t component_max, norm_max, n_listed, n_scan;
};

// 2^(12 - e) for a largest component of 2^e: rows up to 16 times as large stay inside the half's range
__device__ inline float near_scale(uint32_t component_max) {
    const int e = (int)(component_max >> 23) - 127;
    const int s = component_max == 0u ? 0 : 12 - e;
    return __uint_as_float((uint32_t)(127 + (s < -100 ? -100 : s > 100 ? 100 : s)) << 23);
}
// bound of |v_computed - v_exact|, in scaled units; xn, cn: |x'|, largest |c'|
__device__ inline float near_error(int d, float xn, float cn) {
    const float sums = (4.f * (float)d + 40.f) * 5.9604645e-08f + 3.8146973e-06f;
    return (9.8632813e-04f + sums) * xn * cn + sums * 0.5f * cn * cn + __builtin_sqrtf((float)d) * 3.1e-08f * (xn + cn);
}

__global__ void __launch_bounds__(256)
centre_mean_kernel(const float* __restrict__ C, int k, int d, float* __restrict__ mean) {
    // threads along the components; the workgroups share the centres out.  Any mean serves: its rounding decides nothing
    for (int t = threadIdx.x; t < d; t += blockDim.x) {
        float sum = 0.f;
#pragma unroll 8
        for (int c = blockIdx.x; c < k; c += gridDim.x) {
            const float v = C[(size_t)c * d + t];
            sum += __builtin_fabsf(v) < 1e30f ? v : 0.f;
        }
        atomicAdd(&mean[t], sum / (float)k);
    }
}

// norms[c] = |c'|^2, or -1 for a centre with components that are no moderate numbers, which is no part of the product.  One with a component
// that is not finite is at no finite distance, hence never the nearest.  One that is finite can be: the largest norm is then infinite,
// so is the error of a value, and every row compares all centres.
__global__ void __launch_bounds__(1024)
centre_stats_kernel(const float* __restrict__ C, int k, int d, const float* __restrict__ mean, float* __restrict__ norms, NearStats* __restrict__ stats) {
    // one wave per centre in turn; one addition to the shared maxima per workgroup (one per centre serialises: 230 us for 10,000)
    __shared__ uint32_t s_most[2];
    if (threadIdx.x < 2) s_most[threadIdx.x] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    float most = 0.f, largest = 0.f;
    for (int c = blockIdx.x * 16 + (threadIdx.x >> 6); c < k; c += gridDim.x * 16) {
        float top = 0.f, sum = 0.f;
        bool ok = true;
        for (int t = lane; t < d; t += 64) {
            const float v = C[(size_t)c * d + t] - mean[t];
            ok = ok && __builtin_fabsf(v) < 1e18f;
            top = fmaxf(top, __builtin_fabsf(v));
            sum = __builtin_fmaf(v, v, sum);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) { top = fmaxf(top, __shfl_xor(top, off, kWave)); sum += __shfl_xor(sum, off, kWave); }
        ok = __builtin_amdgcn_ballot_w64(!ok) == 0;
        if (lane == 0) norms[c] = ok ? sum : -1.f;
        if (ok) { most = fmaxf(most, top); largest = fmaxf(largest, sum); }
        else {
            bool finite = true;
            for (int t = lane; t < d; t += 64) finite = finite && __builtin_fabsf(C[(size_t)c * d + t]) <= 3.4028235e38f;
            if (__builtin_amdgcn_ballot_w64(!finite) == 0) largest = __builtin_inff();
        }
    }
    if (lane == 0) { atomicMax(&s_most[0], __float_as_uint(most)); atomicMax(&s_most[1], __float_as_uint(largest)); }
    __syncthreads();
    if (threadIdx.x == 0) { atomicMax(&stats->component_max, s_most[0]); atomicMax(&stats->norm_max, s_most[1]); }
}

// X[rows][d] - mean, scaled, in half, slice by slice: [dp / 16][rows_pad][16]; zeros past the matrix.  One thread per 8 components.
// norms (centres only): a centre without one gets zeros, and start[c] = -|c'|^2 / 2 in scaled units (never the largest for those and the padding).
__global__ void __launch_bounds__(256)
near_halves_kernel(const float* __restrict__ X, size_t rows, size_t rows_pad, int d, int dp, const float* __restrict__ mean,
                   const NearStats* __restrict__ stats, const float* __restrict__ norms, float* __restrict__ start, _Float16* __restrict__ out) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t per_row = (uint32_t)dp / 8u;
    const size_t row = t / per_row;
    const int k0 = (int)(t - row * per_row) * 8;
    if (row >= rows_pad) return;
    const float scale = near_scale(stats->component_max);
    const bool ok = row < rows && (!norms || norms[row] >= 0.f);
    half8 h;
    if (ok && k0 + 8 <= d && (d & 3) == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0) {
        const float4 a = reinterpret_cast<const float4*>(X + row * d + k0)[0], b = reinterpret_cast<const float4*>(X + row * d + k0)[1];
        const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int u = 0; u < 8; ++u) h[u] = (_Float16)((v[u] - mean[k0 + u]) * scale);
    } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) h[u] = ok && k0 + u < d ? (_Float16)((X[row * d + k0 + u] - mean[k0 + u]) * scale) : (_Float16)0.f;
    }
    *reinterpret_cast<half8*>(out + ((size_t)(k0 / 16) * rows_pad + row) * 16 + (k0 % 16)) = h;
    if (start && k0 == 0) start[row] = ok ? -0.5f * norms[row] * scale * scale : -3.0e38f;
}

// the larger of two numbers in one instruction (the compiler first quiets one that was made from bits, with another)
__device__ inline float larger(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// One wave per 32 NB rows, four waves per workgroup, and a share of the centres ("split").  v_mfma_f32_32x32x16_f16: rows of a block
// are centres, columns data rows, so a lane holds 16 centres' values of one data row; the accumulator starts at -|c'|^2 / 2.  A value's
// place among the lane's 16 goes into its low four bits; two instructions more keep the largest and the second largest.
// The workgroup stages 64 centres at a time in the LDS, two buffers, one barrier; the stage after next travels in registers.  (Read by every
// wave from the caches instead, 500,000 rows against 10,000 centres wait 60 % of 1.7 ms for them.)
// Bound by issue: the 50 vector instructions per 16 x 64 values and the products (32 cycles each) share a SIMD, and add up.
template <int STEPS, int NB, bool EMIT>
__global__ void __launch_bounds__(kNearThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
near_kernel(const _Float16* __restrict__ Xh, size_t rows_pad, size_t n_rows, const _Float16* __restrict__ Ch, int k_pad,
            const float* __restrict__ start, int splits, uint4* __restrict__ part, const uint2* __restrict__ listed, const NearStats* __restrict__ stats,
            uint32_t* __restrict__ found) {
    constexpr int kWaves = kNearThreads / 64, PER = STEPS / 2;           // 16-byte pieces a thread brings per stage
    static_assert(STEPS % 2 == 0, "every thread brings whole pieces");
    __shared__ __attribute__((aligned(16))) _Float16 s_c[2][STEPS][64 * 16];
    __shared__ __attribute__((aligned(16))) float s_start[2][64];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t count = EMIT ? (size_t)stats->n_listed : n_rows;
    const int n_stages = k_pad / 64;
    const size_t n_tiles = (count + kWaves * 32 * NB - 1) / (kWaves * 32 * NB);         // of a workgroup
    if constexpr (EMIT) {              // as many splits as the listed rows leave workgroups for
        splits = n_tiles > 0 && gridDim.x > n_tiles ? (int)(gridDim.x / n_tiles) : 1;
        splits = splits < n_stages / 2 ? splits : (n_stages / 2 > 0 ? n_stages / 2 : 1);
    }
    for (size_t job = blockIdx.x; job < n_tiles * (size_t)splits; job += gridDim.x) {
        const size_t tile = (job / (uint32_t)splits) * kWaves + (uint32_t)wave;
        const uint32_t split = (uint32_t)(job % (uint32_t)splits);
        const int s0 = (int)((long long)n_stages * split / splits), s1 = (int)((long long)n_stages * (split + 1) / splits);
        half8 pre[PER];
        float4 pre_start = make_float4(0.f, 0.f, 0.f, 0.f);
        auto fetch = [&](int stage) __attribute__((always_inline)) {
            stage = stage < s1 ? stage : s1 - 1;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int p = tid + kNearThreads * i, sl = p >> 7, r = p & 127;
                pre[i] = *reinterpret_cast<const half8*>(Ch + ((size_t)sl * k_pad + (size_t)stage * 64) * 16 + r * 8);
            }
            if (tid < 16) pre_start = reinterpret_cast<const float4*>(start + stage * 64)[tid];
        };
        auto stash = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int p = tid + kNearThreads * i, sl = p >> 7, r = p & 127;
                *reinterpret_cast<half8*>(&s_c[buf][sl][split_piece_at(r >> 1, r & 1)]) = pre[i];
            }
            if (tid < 16) reinterpret_cast<float4*>(s_start[buf])[tid] = pre_start;
        };
        fetch(s0);
        half8 B[NB][STEPS];
        float limit[NB];
        auto place = [&](int b) { return tile * (32 * NB) + 32 * b + l32; };
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            size_t row = place(b) < rows_pad ? place(b) : rows_pad - 1;
            limit[b] = 0.f;
            if constexpr (EMIT) {
                const uint2 e = listed[place(b) < count ? place(b) : count - 1];
                row = e.x;
                limit[b] = place(b) < count ? __uint_as_float(e.y) : 3.4e38f;
            }
#pragma unroll
            for (int s = 0; s < STEPS; ++s) B[b][s] = *reinterpret_cast<const half8*>(Xh + ((size_t)s * rows_pad + row) * 16 + half * 8);
        }
        float m1[NB], m2[NB];
        int at[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) { m1[b] = -3.3e38f; m2[b] = -3.3e38f; at[b] = 0; }
        auto look = [&](const floatx16& acc, auto b_tag, int blk) __attribute__((always_inline)) {
            constexpr int b = decltype(b_tag)::value;
            if constexpr (EMIT) {
                float mx = acc[0];
#pragma unroll
                for (int v = 1; v < 16; ++v) mx = fmaxf(mx, acc[v]);
                if (__builtin_amdgcn_ballot_w64(mx >= limit[b]) == 0) return;
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (acc[v] >= limit[b]) {
                        uint32_t* mine = found + place(b) * (kNearList + 1);
                        const uint32_t slot = atomicAdd(mine, 1u);
                        if (slot < (uint32_t)kNearList) mine[1 + slot] = (uint32_t)(blk * 32 + 8 * (v / 4) + 4 * half + (v % 4));
                    }
            } else {
                const float before = m1[b];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float f = __uint_as_float((__float_as_uint(acc[v]) & ~15u) | (uint32_t)v);
                    m2[b] = __builtin_amdgcn_fmed3f(m1[b], m2[b], f);
                    m1[b] = larger(m1[b], f);
                }
                at[b] = m1[b] != before ? blk : at[b];
            }
        };
        stash(0);
        fetch(s0 + 1);
        __syncthreads();
        for (int st = s0; st < s1; ++st) {
            const int buf = (st - s0) & 1;
            stash(buf ^ 1);                    // its last readers passed the barrier that ended the stage before
            fetch(st + 2);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                floatx16 init, acc[NB];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 h4 = *reinterpret_cast<const float4*>(&s_start[buf][h * 32 + 8 * g + 4 * half]);
                    init[4 * g] = h4.x; init[4 * g + 1] = h4.y; init[4 * g + 2] = h4.z; init[4 * g + 3] = h4.w;
                }
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    const half8 A = *reinterpret_cast<const half8*>(&s_c[buf][s][split_piece_at(h * 32 + l32, half)]);
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, B[b][s], s == 0 ? init : acc[b], 0, 0, 0);
                }
                static_for<NB>([&](auto b_tag) __attribute__((always_inline)) { look(acc[decltype(b_tag)::value], b_tag, st * 2 + h); });
            }
            __syncthreads();
        }
        if constexpr (!EMIT) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                float norm = 0.f;
#pragma unroll
                for (int s = 0; s < STEPS; ++s)
#pragma unroll
                    for (int u = 0; u < 8; ++u) norm = __builtin_fmaf((float)B[b][s][u], (float)B[b][s][u], norm);
                norm += __shfl_xor(norm, 32, kWave);
                const uint32_t v = __float_as_uint(m1[b]) & 15u;
                const int mine = at[b] * 32 + 8 * (int)(v / 4) + 4 * half + (int)(v % 4);
                const float o1 = __shfl_xor(m1[b], 32, kWave), o2 = __shfl_xor(m2[b], 32, kWave);
                const int other = __shfl_xor(mine, 32, kWave);
                const bool take = o1 > m1[b];
                const float first = take ? o1 : m1[b], second = fmaxf(take ? m1[b] : o1, fmaxf(m2[b], o2));
                if (half == 0 && place(b) < n_rows)
                    part[(size_t)split * n_rows + place(b)] = make_uint4(__float_as_uint(first), __float_as_uint(second), (uint32_t)(take ? other : mine), __float_as_uint(norm));
            }
        }
    }
}

__global__ void __launch_bounds__(1024)
near_decide_kernel(const uint4* __restrict__ part, size_t n_rows, int splits, int d, int k, NearStats* __restrict__ stats,
                   int32_t* __restrict__ labels, uint2* __restrict__ listed, uint32_t* __restrict__ found, uint32_t* __restrict__ scan) {
    __shared__ uint32_t s_n[2];            // places in the two lists are taken for the whole workgroup at once
    if (threadIdx.x < 2) s_n[threadIdx.x] = 0u;
    __syncthreads();
    const size_t row = (size_t)blockIdx.x * 1024 + threadIdx.x;
    const int lane = threadIdx.x & 63;
    bool list = false, all = false;
    float limit = 0.f;
    if (row < n_rows) {
        float first = -3.4e38f, second = -3.4e38f, norm = 0.f;
        uint32_t at = 0;
        for (int s = 0; s < splits; ++s) {
            const uint4 p = part[(size_t)s * n_rows + row];
            const float f = __uint_as_float(p.x), g = __uint_as_float(p.y);
            second = fmaxf(second, fmaxf(g, fminf(f, first)));
            if (f > first) { first = f; at = p.z; }
            norm = __uint_as_float(p.w);
        }
        const float scale = near_scale(stats->component_max);
        const float cn = __builtin_sqrtf(__uint_as_float(stats->norm_max)) * scale * 1.0001f, xn = __builtin_sqrtf(norm) * 1.001f;
        const float error = near_error(d, xn, cn);
        // (not-a-number fails every comparison: such a row looks at all centres, as one does that no finite centre was found for; so do all
        // rows where the squares of the centres' components leave the range of a float: below it, or past it and the error with them)
        all = !(__uint_as_float(stats->component_max) > 1.0e-15f) || !(xn < 1.0e18f) || !(error < 1.0e30f) || !(first > -2.9e38f) || at >= (uint32_t)k;
        limit = first - 2.f * error - __builtin_fabsf(first) * 2.0e-6f;
        list = !all && !(second < limit);
        if (!all && !list) labels[row] = (int32_t)at;
    }
    const unsigned long long ml = __builtin_amdgcn_ballot_w64(list), ma = __builtin_amdgcn_ballot_w64(all), below = (1ull << lane) - 1ull;
    uint32_t at_list = 0, at_all = 0;
    if (lane == 0) {
        if (ml != 0) at_list = atomicAdd(&s_n[0], (uint32_t)__popcll(ml));
        if (ma != 0) at_all = atomicAdd(&s_n[1], (uint32_t)__popcll(ma));
    }
    at_list = (uint32_t)__builtin_amdgcn_readfirstlane((int)at_list);
    at_all = (uint32_t)__builtin_amdgcn_readfirstlane((int)at_all);
    __syncthreads();
    if (threadIdx.x == 0) {
        s_n[0] = s_n[0] ? atomicAdd(&stats->n_listed, s_n[0]) : 0u;
        s_n[1] = s_n[1] ? atomicAdd(&stats->n_scan, s_n[1]) : 0u;
    }
    __syncthreads();
    if (list) {
        const size_t slot = s_n[0] + at_list + (uint32_t)__popcll(ml & below);
        listed[slot] = make_uint2((uint32_t)row, __float_as_uint(limit));
        found[slot * (kNearList + 1)] = 0u;
    }
    if (all) scan[s_n[1] + at_all + (uint32_t)__popcll(ma & below)] = (uint32_t)row;
}

// float64 squared distance, components in ascending order, one multiply and one add each
__device__ inline double near_distance(const float* __restrict__ x, const float* __restrict__ c, int d, bool wide) {
    double dist = 0.0;
    int t = 0;
    if (wide)
        for (; t + 4 <= d; t += 4) {
            const float4 a = *reinterpret_cast<const float4*>(x + t), b = *reinterpret_cast<const float4*>(c + t);
            double e = (double)a.x - (double)b.x; dist += e * e;
            e = (double)a.y - (double)b.y; dist += e * e;
            e = (double)a.z - (double)b.z; dist += e * e;
            e = (double)a.w - (double)b.w; dist += e * e;
        }
    for (; t < d; ++t) { const double e = (double)x[t] - (double)c[t]; dist += e * e; }
    return dist;
}

// The listed rows: 16 lanes per row, one centre each
__global__ void __launch_bounds__(256)
near_exact_kernel(const float* __restrict__ X, const float* __restrict__ C, int d, int wide, const uint2* __restrict__ listed, const uint32_t* __restrict__ found,
                  NearStats* __restrict__ stats, int32_t* __restrict__ labels, uint32_t* __restrict__ scan) {
    const uint32_t n = stats->n_listed, l16 = threadIdx.x & 15u;
    const uint32_t rounds = (n + 15u) / 16u;
    for (uint32_t r = blockIdx.x; r < rounds; r += gridDim.x) {
        const uint32_t i = r * 16u + (threadIdx.x >> 4);
        double best = __longlong_as_double(0x7FF0000000000000ll);
        uint32_t arg = 0xFFFFFFFFu, count = 0;
        size_t row = 0;
        if (i < n) {
            row = listed[i].x;
            const uint32_t* mine = found + (size_t)i * (kNearList + 1);
            count = mine[0];
            if (count <= (uint32_t)kNearList && l16 < count) {
                const uint32_t c = mine[1 + l16];
                const double dist = near_distance(X + row * d, C + (size_t)c * d, d, wide != 0);
                if (dist < best) { best = dist; arg = c; }
            }
        }
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) {
            const double ob = __shfl_xor(best, off, kWave);
            const uint32_t oa = (uint32_t)__shfl_xor((int)arg, off, kWave);
            if (ob < best || (ob == best && oa < arg)) { best = ob; arg = oa; }
        }
        if (i < n && l16 == 0) {
            if (count <= (uint32_t)kNearList && arg != 0xFFFFFFFFu) labels[row] = (int32_t)arg;
            else scan[atomicAdd(&stats->n_scan, 1u)] = (uint32_t)row;
        }
    }
}

// Rows that compare all centres: one workgroup per row
__global__ void __launch_bounds__(256)
near_scan_kernel(const float* __restrict__ X, const float* __restrict__ C, int k, int d, int wide, const uint32_t* __restrict__ scan,
                 const NearStats* __restrict__ stats, int32_t* __restrict__ labels) {
    __shared__ double s_best[256];
    __shared__ int s_arg[256];
    const int tid = threadIdx.x;
    const uint32_t n = stats->n_scan;
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
        const size_t row = scan[i];
        double best = __longlong_as_double(0x7FF0000000000000ll);
        int arg = 0x7FFFFFFF;
        for (int c = tid; c < k; c += 256) {
            const double dist = near_distance(X + row * d, C + (size_t)c * d, d, wide != 0);
            if (dist < best) { best = dist; arg = c; }
        }
        s_best[tid] = best; s_arg[tid] = arg;
        __syncthreads();
        for (int off = 128; off > 0; off >>= 1) {
            if (tid < off) {
                const double ob = s_best[tid + off];
                const int oa = s_arg[tid + off];
                if (ob < s_best[tid] || (ob == s_best[tid] && oa < s_arg[tid])) { s_best[tid] = ob; s_arg[tid] = oa; }
            }
            __syncthreads();
        }
        if (tid == 0) labels[row] = s_arg[0] < k ? s_arg[0] : 0;             // no finite distance: stay in range
        __syncthreads();
    }
}

// Places of the step's buffers inside a workspace of `bytes` bytes.
struct NearLayout {
    int dp, splits;
    size_t rows_pad, k_pad;
    size_t xh, ch, start, norms, mean, stats, part, listed, found, scan, bytes;
};
inline int near_blocks(int dp) { return dp > 96 ? 3 : 4; }       // blocks of 32 rows per wave: as many as the registers hold
inline bool near_dims(int d) { return d >= 1 && d <= 128; }
inline NearLayout near_layout(size_t n_rows, int k, int d) {
    NearLayout L{};
    L.dp = (d + 31) / 32 * 32;
    L.rows_pad = (n_rows + 127) / 128 * 128;
    L.k_pad = ((size_t)k + 63) / 64 * 64;
    // few rows: the centres are split among workgroups, so that every compute unit has two; two stages of centres or more each
    const size_t tile = (size_t)(kNearThreads / 64) * 32 * near_blocks(L.dp), tiles = (n_rows + tile - 1) / tile;
    size_t splits = (512 + tiles - 1) / tiles;
    const size_t most = L.k_pad / 128 > 0 ? L.k_pad / 128 : 1;
    splits = splits > most ? most : splits;
    L.splits = (int)(splits > 16 ? 16 : splits);
    size_t at = 0;
    auto take = [&](size_t bytes) { size_t o = at; at = align_up(at + bytes); return o; };
    L.mean = take((size_t)d * 4);
    L.stats = take(sizeof(NearStats));
    L.xh = take(L.rows_pad * L.dp * 2);
    L.ch = take(L.k_pad * L.dp * 2);
    L.start = take(L.k_pad * 4);
    L.norms = take((size_t)k * 4);
    L.part = take((size_t)L.splits * n_rows * 16);
    L.listed = take(n_rows * 8);
    L.found = take(n_rows * (kNearList + 1) * 4);
    L.scan = take(n_rows * 4);
    L.bytes = at;
    return L;
}

template <int STEPS, int NB>
int launch_near(const NearLayout& L, unsigned char* ws, size_t n_rows, hipStream_t st, bool emit) {
    const _Float16* xh = (const _Float16*)(ws + L.xh);
    const _Float16* ch = (const _Float16*)(ws + L.ch);
    const float* start = (const float*)(ws + L.start);
    const NearStats* stats = (const NearStats*)(ws + L.stats);
    const size_t tile = (size_t)(kNearThreads / 64) * 32 * NB, blocks = (n_rows + tile - 1) / tile * L.splits;
    if (!emit)
        hipLaunchKernelGGL((near_kernel<STEPS, NB, false>), dim3((unsigned)blocks), dim3(kNearThreads), 0, st, xh, L.rows_pad, n_rows, ch, (int)L.k_pad,
                           start, L.splits, (uint4*)(ws + L.part), (const uint2*)nullptr, stats, (uint32_t*)nullptr);
    else
        hipLaunchKernelGGL((near_kernel<STEPS, NB, true>), dim3(512), dim3(kNearThreads), 0, st, xh, L.rows_pad, n_rows, ch, (int)L.k_pad,
                           start, 1, (uint4*)nullptr, (const uint2*)(ws + L.listed), stats, (uint32_t*)(ws + L.found));
    HIP_TRY(hipGetLastError());
    return IVFPQ_OK;
}

// labels[i] = the nearest of k centres for n_rows rows (below 2^31), in `ws` (near_layout bytes)
int nearest_by_halves(unsigned char* ws, const float* X, size_t n_rows, const float* C, int k, int d, int32_t* labels, hipStream_t st) {
    const NearLayout L = near_layout(n_rows, k, d);
    float* mean = (float*)(ws + L.mean);
    NearStats* stats = (NearStats*)(ws + L.stats);
    float* norms = (float*)(ws + L.norms);
    const size_t clear = (L.xh - L.mean) / 4;                  // mean and statistics
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((clear + 255) / 256)), dim3(256), 0, st, (uint32_t*)(ws + L.mean), clear, 0u);
    hipLaunchKernelGGL(centre_mean_kernel, dim3(128), dim3(d <= 64 ? 64 : 128), 0, st, C, k, d, mean);
    hipLaunchKernelGGL(centre_stats_kernel, dim3(std::min(256, (k + 15) / 16)), dim3(1024), 0, st, C, k, d, mean, norms, stats);
    auto halves = [&](const float* M, size_t rows, size_t rows_pad, const float* nm, float* start, size_t out) {
        const size_t threads = rows_pad * (L.dp / 8);
        hipLaunchKernelGGL(near_halves_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, M, rows, rows_pad, d, L.dp, mean, stats, nm, start,
                           (_Float16*)(ws + out));
    };
    halves(C, (size_t)k, L.k_pad, norms, (float*)(ws + L.start), L.ch);
    halves(X, n_rows, L.rows_pad, nullptr, nullptr, L.xh);
    HIP_TRY(hipGetLastError());
    auto near = [&](bool emit) -> int {
        switch (L.dp) {
            case 32: return launch_near<2, 4>(L, ws, n_rows, st, emit);
            case 64: return launch_near<4, 4>(L, ws, n_rows, st, emit);
            case 96: return launch_near<6, 4>(L, ws, n_rows, st, emit);
            default: return launch_near<8, 3>(L, ws, n_rows, st, emit);
        }
    };
    if (int s = near(false)) return s;
    uint2* listed = (uint2*)(ws + L.listed);
    uint32_t* found = (uint32_t*)(ws + L.found);
    uint32_t* scan = (uint32_t*)(ws + L.scan);
    hipLaunchKernelGGL(near_decide_kernel, dim3((unsigned)((n_rows + 1023) / 1024)), dim3(1024), 0, st, (const uint4*)(ws + L.part), n_rows, L.splits, d, k, stats,
                       labels, listed, found, scan);
    HIP_TRY(hipGetLastError());
    if (int s = near(true)) return s;
    const int wide = d % 4 == 0 && ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(C)) & 15) == 0;
    hipLaunchKernelGGL(near_exact_kernel, dim3(2048), dim3(256), 0, st, X, C, d, wide, listed, found, stats, labels, scan);
    hipLaunchKernelGGL(near_scan_kernel, dim3(1024), dim3(256), 0, st, X, C, k, d, wide, scan, stats, labels);
    HIP_TRY(hipGetLastError());
    return IVFPQ_OK;
}

}  // namespace
