// Eq. (1) for the vectors that the matrix-core filter lists (ivfpq_scan_filter.hip).  Compiled once per table dtype,
// IVFPQ_CANDIDATE_LUT.
#include <hip/hip_runtime.h>

#include "ivfpq_hip_util.hpp"
#include "ivfpq_lds_util.hpp"
#include "ivfpq_scan_filter.hpp"

using namespace ivfpq;

namespace {

constexpr int kCandidateThreads = 1024;
constexpr uint32_t kParts = 4;       // tickets per query and workgroup: the lists differ in length, and a workgroup has few queries
constexpr uint32_t kCandidateBlocks = 256;
// Workgroups that share a query's list, a power of two: few queries with long lists would leave most of the chip idle
// (search of 400 / 100 queries, k = 100, 30 of 100 lists of 1,000, four waves a query: 320 / 300 us; shared: 164 / 105).
inline uint32_t candidate_share(int nq) {
    uint32_t s = 1;
    while (s < 64u && (uint64_t)s * (uint32_t)nq < 2048u) s *= 2;
    return s;
}

// A table entry as a lookup returns it: stored in the table's type and read back.
template <int LUT>
__device__ __forceinline__ float stored_entry(float f, const Fp8Params fp8, int hi_v, int half_ulp, int mask) {
    if constexpr (LUT == IVFPQ_LUT_FP32) {
        return f;
    } else if constexpr (LUT == IVFPQ_LUT_FP16) {
        return __half2float(__ushort_as_half((unsigned short)half_bits_from_f32(f)));
    } else {
        // decode(encode(f)) on the FP32 pattern: clamp to the format's range, add half an 8-bit ulp (nothing to truncate),
        // drop the bits below the mantissa.  The smallest value is a multiple of the ulp, so the code's offset cancels.
        int b;
        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(b) : "v"(__float_as_int(f)), "s"(fp8.lo), "v"(hi_v));
        return __int_as_float((b + half_ulp) & mask);
    }
}

// One wave per query at a time, one lane per listed vector: its table entries are formed from the codebooks (in the LDS, in
// fp32, for the whole life of the workgroup), the query and the centroid of its cluster, rounded to the table's type and added
// in ascending order, as a table scan would.
template <int LUT, int BITS, int M>
__global__ void __launch_bounds__(kCandidateThreads)
candidate_kernel(const float* __restrict__ queries, FilterArgs a, uint32_t share) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int KSUB = 1 << BITS;
    constexpr int G = (BITS % 8 == 0) ? 8 : (BITS % 4 == 0) ? 4 : (BITS % 2 == 0) ? 2 : 1;
    constexpr int SPG = 32 / G, WPG = BITS / G;                 // the shortest run of codes that is whole words
    const int n_floats = a.d * KSUB;
    uint32_t* ticket = reinterpret_cast<uint32_t*>(smem + (size_t)n_floats * 4);
    for (int i = threadIdx.x; i < n_floats / 4; i += kCandidateThreads)
        reinterpret_cast<float4*>(smem)[i] = reinterpret_cast<const float4*>(a.codebooks)[i];
    if (threadIdx.x == 0) *ticket = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    int hi_v = a.fp8.hi;
    asm volatile("" : "+v"(hi_v));
    constexpr int SH = LUT == IVFPQ_LUT_FP8_E5M3 || LUT == IVFPQ_LUT_FP8_E4M4 ? Fp8Format<LUT == IVFPQ_LUT_FP8_E4M4 ? IVFPQ_LUT_FP8_E4M4 : IVFPQ_LUT_FP8_E5M3>::shift : 20;
    const int half_ulp = a.truncate ? 0 : 1 << (SH - 1), mask = ~((1 << SH) - 1);
    for (;;) {
        uint32_t t = 0;
        if (lane == 0) t = atomicAdd(ticket, 1u);
        t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
        const uint32_t parts = kParts * share, part = t % kParts + kParts * (blockIdx.x % share), q = t / kParts * (gridDim.x / share) + blockIdx.x / share;
        if (q >= (uint32_t)a.nq) break;
        const uint32_t n0 = a.starts[q], n = a.counts[q];
        if (n <= n0) continue;
        const uint4* pairs = a.pairs + (size_t)q * a.n_probes;
        const size_t row = (size_t)q * a.stride + pairs[1].w;
        const float* qv = queries + (size_t)q * a.d;
        for (uint32_t base = n0 + 64u * part; base < n; base += 64u * parts) {
            const uint32_t i = base + (uint32_t)lane, ii = i < n ? i : n - 1u;
            const uint32_t pos = a.row_pos[row + ii], probe = a.row_key[row + ii];
            const uint4 pair = pairs[probe];
            const uint32_t v = pos - pair.w;
            const unsigned char* code = a.codes + ((size_t)pair.z + (v >> 6)) * 64 * a.code_bytes;
            const float* c = a.centroids + (size_t)pair.x * a.d;
            float acc = 0.f;
            // Adds the entries of the codes in w[0 .. NW), sub-spaces from sub0 on, four at a time: the four codewords' LDS
            // reads and the next four sub-spaces' centroid components are under way together before any is used.  c_now: the centroid
            // components of the first four; on return those of the four that follow.
            float4 c_now[M];
#pragma unroll
            for (int v = 0; v < M; ++v) c_now[v] = reinterpret_cast<const float4*>(c)[v];
            auto add = [&](const uint32_t* w, auto words_tag, int sub0) __attribute__((always_inline)) {
                constexpr int NW = decltype(words_tag)::value, NS = NW / WPG * SPG;
                const unsigned char* book = smem + (size_t)sub0 * (KSUB * M * 4);
                static_for<NS / 4>([&](auto b_tag) __attribute__((always_inline)) {
                    constexpr int B = decltype(b_tag)::value;
                    const int at = sub0 + 4 * B;                         // first of the four sub-spaces
                    float cb[4][M];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int s = B * 4 + u, bit = s * BITS, wi = bit >> 5, sh = bit & 31;
                        uint32_t cd;
                        if (sh + BITS > 32) cd = __builtin_amdgcn_alignbit(w[wi + 1 < NW ? wi + 1 : wi], w[wi], sh) & (uint32_t)(KSUB - 1);
                        else cd = (w[wi] >> sh) & (uint32_t)(KSUB - 1);
                        const unsigned char* e = book + cd * (uint32_t)(M * 4) + s * (KSUB * M * 4);
                        if constexpr (M == 2) { const float2 x = *reinterpret_cast<const float2*>(e); cb[u][0] = x.x; cb[u][1] = x.y; }
                        else { const float4 x = *reinterpret_cast<const float4*>(e); cb[u][0] = x.x; cb[u][1] = x.y; cb[u][2] = x.z; cb[u][3] = x.w; }
                    }
                    float4 c_next[M];
                    const int after = at + 4 < a.pq_dim ? at + 4 : 0;
#pragma unroll
                    for (int v = 0; v < M; ++v) c_next[v] = reinterpret_cast<const float4*>(c + after * M)[v];
                    float qq[4 * M];
#pragma unroll
                    for (int v = 0; v < 4 * M; ++v) qq[v] = qv[at * M + v];
                    __builtin_amdgcn_sched_barrier(0);
                    float r[4 * M];
#pragma unroll
                    for (int v = 0; v < M; ++v) {
                        r[4 * v] = qq[4 * v] - c_now[v].x; r[4 * v + 1] = qq[4 * v + 1] - c_now[v].y;
                        r[4 * v + 2] = qq[4 * v + 2] - c_now[v].z; r[4 * v + 3] = qq[4 * v + 3] - c_now[v].w;
                        c_now[v] = c_next[v];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) acc += stored_entry<LUT>(lut_entry<M>(cb[u], r + u * M), a.fp8, hi_v, half_ulp, mask);
                    __builtin_amdgcn_sched_barrier(0);
                });
            };
            const int n_words = a.code_bytes / 4;
            if (a.chunk_width == 16 && WPG == 1) {
                for (int w0 = 0; w0 < n_words; w0 += 4) {
                    const uint4 x = *reinterpret_cast<const uint4*>(code + ((w0 >> 2) * 64 + (int)(v & 63u)) * 16);
                    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
                    if constexpr (WPG == 1) add(w, std::integral_constant<int, 4>{}, w0 * SPG);
                }
            } else {
                for (int w0 = 0; w0 < n_words; w0 += WPG) {
                    uint32_t w[WPG];
#pragma unroll
                    for (int u = 0; u < WPG; ++u) {
                        const int wi = w0 + u;
                        w[u] = *reinterpret_cast<const uint32_t*>(code + (a.chunk_width == 16 ? ((wi >> 2) * 64 + (int)(v & 63u)) * 16 + (wi & 3) * 4
                                                                                             : (wi * 64 + (int)(v & 63u)) * 4));
                    }
                    add(w, std::integral_constant<int, WPG>{}, w0 / WPG * SPG);
                }
            }
            if (i < n) a.row_key[row + i] = __float_as_uint(acc);
        }
    }
}

}  // namespace

template <int LUT>
int ivfpq::launch_candidates_lut(const FilterArgs& a, hipStream_t st) {
    auto go = [&](auto kernel) -> int {
        if (int s = allow_full_lds(kernel)) return s;
        hipLaunchKernelGGL(kernel, dim3(kCandidateBlocks), dim3(kCandidateThreads), candidate_lds_bytes(a.bits, a.d), st, a.queries, a, candidate_share(a.nq));
        HIP_TRY(hipGetLastError());
        return IVFPQ_OK;
    };
    switch (a.bits * 8 + a.m) {
        case 8 * 8 + 2: return go(candidate_kernel<LUT, 8, 2>);
        case 8 * 8 + 4: return go(candidate_kernel<LUT, 8, 4>);
        case 7 * 8 + 2: return go(candidate_kernel<LUT, 7, 2>);
        case 6 * 8 + 2: return go(candidate_kernel<LUT, 6, 2>);
        case 5 * 8 + 2: return go(candidate_kernel<LUT, 5, 2>);
        case 4 * 8 + 2: return go(candidate_kernel<LUT, 4, 2>);
        case 4 * 8 + 4: return go(candidate_kernel<LUT, 4, 4>);
        default: return fail(IVFPQ_EUNSUPPORTED, "internal: no candidate kernel for %d-bit codes of %d components", a.bits, a.m);
    }
}

template int ivfpq::launch_candidates_lut<IVFPQ_CANDIDATE_LUT>(const FilterArgs&, hipStream_t);
#if IVFPQ_CANDIDATE_LUT == 0
size_t ivfpq::candidate_lds_bytes(int bits, int d) { return ((size_t)d << bits) * 4 + 16; }
#endif
