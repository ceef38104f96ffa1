// The filtered scan of large batches on the matrix cores.
//
// Of the vectors of a query's other probes only those with R <= bound (the k-th smallest R of its nearest probe) matter,
// one in a few hundred.  R is the sum of table entries F_j = |cb_j[y_j] - r_j|^2 in the table's storage type, so
// R >= (1 - e) |r - y|^2 less a little (e: the largest relative loss of a stored entry; y: the vector's decoded
// residual, r: the query's), and |r - y|^2 = |r|^2 - 2 r.y + |y|^2 for all pairs of a cluster and all its vectors is a
// matrix product.  This kernel forms it in bf16 with the rounding bounded (filter threshold, below) and lists every vector
// that could have R <= bound; candidate_kernel (ivfpq_candidates.hip) then makes the sum of Eq. (1) for the listed ones alone,
// entry by entry in the table's type and order.  The survivors, hence all results, are those of a scan of every vector.
//
// A table lookup costs the vector ALU and the LDS several cycles per vector, query and sub-space; here the codeword of a
// (vector, sub-space) is fetched from the LDS once for up to 64 queries, straight into the matrix operand of the lane that
// holds it, and the query's share is a fused multiply-add on the matrix cores.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ivfpq_filter_bound.hpp"
#include "ivfpq_hip_util.hpp"
#include "ivfpq_lds_util.hpp"
#include "ivfpq_scan_filter.hpp"

using namespace ivfpq;

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kFilterThreads = 512, kFilterWaves = kFilterThreads / 64;
constexpr int kFilterSteps = kFilterVectors / 32;       // vectors are taken 32 at a time
constexpr int kTurnPitch = 256 + 16;                    // bytes between rows of residuals in the LDS
// a wave's own LDS, in words: rows of residuals in turn, then a word per (step, slot); behind them two thresholds per slot
constexpr int kStartWords = kFilterSteps * 64 * 4 > 16 * kTurnPitch ? kFilterSteps * 64 : 16 * kTurnPitch / 4;
constexpr int kWaveWords = kStartWords + 128;
constexpr float kNever = -3.0e38f, kAlways = 3.0e38f;

// BITS: bits of a code; M: components of a sub-space; STEPS: d / 16.
//
// One wave per work item (up to 64 pairs of a cluster, up to 512 of its vectors), with no barrier after the codebooks are
// in place.  v_mfma_f32_32x32x16_bf16: rows are pairs, columns vectors.  Lane L brings row / column L % 32 and eight
// components; the components are dealt so that half-wave h holds the h-th half of the vector in every operand, i.e. a
// lane decodes the h-th half of its vector's code words, which are consecutive.  The pairs' residuals stay in registers for
// the whole item, the accumulator starts at the pair's threshold, and the largest of a lane's 32 sums against half the
// squared norm of its vector says whether anything passes.
template <int BITS, int M, int STEPS>
struct FilterShape {
    static constexpr int D = 16 * STEPS, SUBS = D / M, KSUB = 1 << BITS;
    static constexpr int WORDS = SUBS * BITS / 32;                 // code words of a vector
    static constexpr bool valid = SUBS * BITS % 64 == 0;           // both halves are whole words
    static constexpr int CB = WORDS * 4;
    static constexpr int CW = (CB % 16 == 0 && CB / 16 <= 4 && (BITS == 4 || BITS == 8 || (BITS == 6 && CB == 48))) ? 16 : 4;
    static constexpr int WPH = WORDS / 2;                          // words of half a vector
    static constexpr int PIECE = CW == 4 ? 1 : (WPH % 4 == 0 ? 4 : 2);     // words of one load
    static constexpr int PIECES = WPH / PIECE;
    static constexpr int E = 2 * M;                                // bytes of a codeword in the LDS
    static constexpr int SPS = 8 / M;                              // sub-spaces of a half-wave and step
    static constexpr int SPH = SUBS / 2;
    static constexpr int H = STEPS / 2;                            // steps before the first test
    static constexpr size_t book_bytes = (size_t)D * KSUB * 2;
};

// A pair of the grouped order, as pair_records_kernel leaves it: {query, slot of the probe, |r|^2, bound}.
// An item, two words of four: {cluster, first pair, number of pairs, number of vectors}, {first vector, first 64-vector group, -, -}.
struct Item {
    uint32_t cluster, first, n_pairs, n_vec, v0, group;
};
__device__ __forceinline__ Item item_of(const uint4 x, const uint4 y) {
    auto uni = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    return Item{uni(x.x), uni(x.y), uni(x.z), uni(x.w), uni(y.x), uni(y.y)};
}

// the sum of a value over lanes L and L ^ 32, in both
__device__ __forceinline__ float sum_of_halves(float v) {
    const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(both[0]) + __uint_as_float(both[1]);
}

// rec: the lane's pair (lane = slot; lanes past the last pair hold the last one).  next_records(): called once, when the item
// after this one has to be known.
template <int BITS, int M, int STEPS, int T, class Next>
__device__ __forceinline__ void filter_item(const FilterArgs& a, uint32_t* bits, const Item item, const uint4 rec, Next next_records) {
    using S = FilterShape<BITS, M, STEPS>;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const uint32_t n_pairs = item.n_pairs, n_vec = item.n_vec;
    const int n_it = (int)((n_vec + 31u) >> 5);

    // the first code words travel while the residuals are formed
    const unsigned char* codes = a.codes + (size_t)item.group * 64 * S::CB;
    uint32_t piece_at[S::PIECES];
#pragma unroll
    for (int p = 0; p < S::PIECES; ++p) {
        const int w = half * S::WPH + p * S::PIECE;
        piece_at[p] = S::CW == 16 ? (uint32_t)(((w >> 2) * 64 + l32) * 16 + (w & 3) * 4) : (uint32_t)((w * 64 + l32) * 4);
    }
    auto load = [&](uint32_t (&w)[S::WPH], int it) __attribute__((always_inline)) {
        it = it < n_it ? it : n_it - 1;
        const unsigned char* base = codes + (size_t)(it >> 1) * 64 * S::CB + (it & 1) * 32 * S::CW;
#pragma unroll
        for (int p = 0; p < S::PIECES; ++p) {
            if constexpr (S::PIECE == 4) {
                const uint4 x = *reinterpret_cast<const uint4*>(base + piece_at[p]);
                w[4 * p] = x.x; w[4 * p + 1] = x.y; w[4 * p + 2] = x.z; w[4 * p + 3] = x.w;
            } else if constexpr (S::PIECE == 2) {
                const uint2 x = *reinterpret_cast<const uint2*>(base + piece_at[p]);
                w[2 * p] = x.x; w[2 * p + 1] = x.y;
            } else {
                w[p] = *reinterpret_cast<const uint32_t*>(base + piece_at[p]);
            }
        }
    };
    uint32_t words_a[S::WPH], words_b[S::WPH], words_c[S::WPH];
    load(words_a, 0);
    load(words_b, 1);

    // Residuals: 16 rows at a time, read whole (a lane two components), rounded to bf16 and turned into the matrix layout through
    // the LDS (the wave's own words; the rows' pitch puts the 16 rows of a 16-byte read on different banks).
    // Read in the matrix layout instead, a row is touched 16 bytes at a time, sixteen times over.
    bf16x8 A[T][STEPS];
    floatx16 C[T];
    float* const starts = reinterpret_cast<float*>(bits + kStartWords);
    {
        unsigned char* const turn = reinterpret_cast<unsigned char*>(bits);
        const bool part = 2 * lane < S::D;
        float2 c = make_float2(0.f, 0.f);
        if (part) c = reinterpret_cast<const float2*>(a.centroids + (size_t)item.cluster * S::D)[lane];
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float2 x[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const uint32_t q = (uint32_t)__builtin_amdgcn_readlane((int)rec.x, t * 32 + h * 16 + r);
                    x[r] = make_float2(0.f, 0.f);
                    if (part) x[r] = reinterpret_cast<const float2*>(a.queries + (size_t)q * S::D)[lane];
                }
                if (part) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const bf16x2_t v = {(__bf16)(x[r].x - c.x), (__bf16)(x[r].y - c.y)};
                        *reinterpret_cast<bf16x2_t*>(turn + r * kTurnPitch + lane * 4) = v;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if ((l32 >> 4) == h) {
                    const unsigned char* mine = turn + (l32 & 15) * kTurnPitch + half * (STEPS * 16);
#pragma unroll
                    for (int s = 0; s < STEPS; ++s) A[t][s] = *reinterpret_cast<const bf16x8*>(mine + s * 16);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
    }
    // Thresholds: lane = row (slot t * 32 + L % 32), both half-waves the same.
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int slot = t * 32 + l32;
        const float rr = __shfl(__uint_as_float(rec.z), slot, 64);
        const uint32_t bnd = (uint32_t)__shfl((int)rec.w, slot, 64);
        // An entry of a table that saturates at `top` loses at most (|r_j| + largest codeword)^2 - top.
        float hidden = 0.f;
        if (a.top < 3.4e38f) {
            auto entry_max = [&](float n2) __attribute__((always_inline)) {          // n2: from components rounded to bf16
                const float x = __builtin_sqrtf(n2 * kRoundedNorm) + a.word_norm_max;
                return x * x * kEntrySlack;
            };
            auto norms = [&](auto sink) __attribute__((always_inline)) {
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    const u32x4_t w = __builtin_bit_cast(u32x4_t, A[t][s]);
#pragma unroll
                    for (int g = 0; g < S::SPS; ++g) {
                        float n2 = 0.f;
#pragma unroll
                        for (int u = 0; u < M / 2; ++u) {
                            const bf16x2_t p = __builtin_bit_cast(bf16x2_t, (uint32_t)w[g * (M / 2) + u]);
                            n2 = __builtin_amdgcn_fdot2_f32_bf16(p, p, n2, false);
                        }
                        sink(n2);
                    }
                }
            };
            float big = 0.f;
            norms([&](float n2) { big = fmaxf(big, n2); });
            if (ballot64(!(entry_max(big) <= a.top)) != 0) {
                norms([&](float n2) { hidden += fmaxf(entry_max(n2) - a.top, 0.f); });
                hidden += __shfl_xor(hidden, 32, 64);
                hidden *= kHiddenSlack;
            }
        }
        // R <= bound implies r.y >= (|r|^2 + |y|^2 - limit) / 2; the product formed here is within eta (|r|^2 + |y|^2) / 2 and
        // the rounding of the threshold's own terms of r.y
        const float limit = __builtin_fmaf(__uint_as_float(bnd), a.scale, a.add) + hidden, wide = limit * (1.f + a.eta * kLimitShare);
        float c = 0.5f * (wide - (1.f - a.eta) * rr);
        // the same for the components of the first H steps alone, whose share of the distance is no more than all of it
        float rr1 = 0.f;
#pragma unroll
        for (int s = 0; s < S::H; ++s) {
            const u32x4_t w = __builtin_bit_cast(u32x4_t, A[t][s]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bf16x2_t p = __builtin_bit_cast(bf16x2_t, (uint32_t)w[u]);
                rr1 = __builtin_amdgcn_fdot2_f32_bf16(p, p, rr1, false);
            }
        }
        rr1 = sum_of_halves(rr1);
        float c1 = 0.5f * (wide - (1.f - a.eta - kSquareLoss) * rr1);
        const bool used = (uint32_t)slot < n_pairs;
        const bool admit = bnd >= 0x7F800000u || !(rr < 1.0e30f);           // no bound, or not a number to compare: every vector passes
        if (!used) c = c1 = kNever;
        else if (admit || !(c < kAlways) || !(c1 < kAlways)) c = c1 = kAlways;
        if (ballot64(admit) != 0) {
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
#pragma unroll
                for (int u = 0; u < 8; ++u) A[t][s][u] = admit ? (__bf16)0.f : A[t][s][u];
        }
        starts[slot] = c1;
        starts[64 + slot] = c - c1;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // register v of a lane: row 8 (v / 4) + 4 (L / 32) + v % 4
    auto rows_of = [&](const float* from, int t, int g) __attribute__((always_inline)) { return *reinterpret_cast<const float4*>(from + t * 32 + 8 * g + 4 * half); };
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 c4 = rows_of(starts, t, g);
            C[t][4 * g] = c4.x; C[t][4 * g + 1] = c4.y; C[t][4 * g + 2] = c4.z; C[t][4 * g + 3] = c4.w;
        }

    const float y_scale = 0.5f * (1.f - a.eta - kSquareLoss);
    uint32_t book0 = (uint32_t)half * (uint32_t)(S::SPH * S::KSUB * S::E);
    asm volatile("" : "+v"(book0));       // opaque: a sub-space's own offset then goes into the read's immediate
    // Codewords of the first H steps of the next 32 vectors, fetched while those of the present ones are multiplied.
    u32x4_t ring[S::H];
    auto fetch = [&](const uint32_t (&w)[S::WPH], auto s_tag) __attribute__((always_inline)) -> u32x4_t {
        constexpr int s = decltype(s_tag)::value;
        uint32_t y[4];
#pragma unroll
        for (int g = 0; g < S::SPS; ++g) {
            const int sub = s * S::SPS + g, bit = sub * BITS, wi = bit >> 5, sh = bit & 31;
            // a code's place in its sub-space's row: for whole bytes and nibbles one dot product with a constant that holds the
            // codeword's size at the code's place extracts, scales and adds
            uint32_t at;
            if constexpr (BITS == 8) {
                at = __builtin_amdgcn_udot4(w[wi], (uint32_t)S::E << sh, book0, false);
            } else if constexpr (BITS == 4) {
                at = __builtin_amdgcn_udot8(w[wi], (uint32_t)S::E << sh, book0, false);
            } else {
                uint32_t code;
                if (sh + BITS > 32) code = __builtin_amdgcn_alignbit(w[wi + 1 < S::WPH ? wi + 1 : wi], w[wi], sh) & (uint32_t)(S::KSUB - 1);
                else code = (w[wi] >> sh) & (uint32_t)(S::KSUB - 1);
                at = code * (uint32_t)S::E + book0;
            }
            const auto x = LdsWord<S::E>::load(at + (uint32_t)(sub * S::KSUB * S::E));
            if constexpr (M == 2) y[g] = x;
            else { y[2 * g] = x.x; y[2 * g + 1] = x.y; }
        }
        return u32x4_t{y[0], y[1], y[2], y[3]};
    };
    static_for<S::H>([&](auto s_tag) __attribute__((always_inline)) { ring[decltype(s_tag)::value] = fetch(words_a, s_tag); });
    auto square = [&](const u32x4_t y, float sum) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bf16x2_t p = __builtin_bit_cast(bf16x2_t, (uint32_t)y[u]);
            sum = __builtin_amdgcn_fdot2_f32_bf16(p, p, sum, false);
        }
        return sum;
    };
    uint32_t met = 0;                 // bit it: vectors 32 it ... have candidates (wave-uniform)
    // 32 vectors: `now` holds their code words, `then` those of the next 32; `later` takes those of the 32 after
    auto round = [&](const uint32_t (&now)[S::WPH], const uint32_t (&then)[S::WPH], uint32_t (&later)[S::WPH], int it) __attribute__((always_inline)) {
        load(later, it + 2);
        floatx16 acc[T];
        float yy = 0.f;
        static_for<S::H>([&](auto s_tag) __attribute__((always_inline)) {
            constexpr int s = decltype(s_tag)::value;
            const bf16x8 B = __builtin_bit_cast(bf16x8, ring[s]);
#pragma unroll
            for (int t = 0; t < T; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[t][s], B, s == 0 ? C[t] : acc[t], 0, 0, 0);
            yy = square(ring[s], yy);
            ring[s] = fetch(then, s_tag);
            // a product keeps the matrix core busy for 32 cycles: the vector instructions and LDS reads go in its shadow
#pragma unroll
            for (int t = 0; t < T; ++t) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 8 / T, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, S::SPS / T, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        const bool real = (uint32_t)(it * 32 + l32) < n_vec;
        auto passes = [&](float need) __attribute__((always_inline)) {
            float mx = kNever;
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc[t][i]);
            return ballot64(mx >= need) != 0;
        };
        auto need_of = [&](float sum) __attribute__((always_inline)) { return real ? sum * y_scale : __uint_as_float(0x7F800000u); };
        // Distances only grow with the components: where no sum of the first half of them passes, the rest is left out.
        if (passes(need_of(sum_of_halves(yy)))) {
            u32x4_t rest[S::H];
            static_for<S::H>([&](auto s_tag) __attribute__((always_inline)) {
                constexpr int s = decltype(s_tag)::value;
                rest[s] = fetch(now, std::integral_constant<int, S::H + s>{});
            });
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 c4 = rows_of(starts + 64, t, g);
                    acc[t][4 * g] += c4.x; acc[t][4 * g + 1] += c4.y; acc[t][4 * g + 2] += c4.z; acc[t][4 * g + 3] += c4.w;
                }
            static_for<S::H>([&](auto s_tag) __attribute__((always_inline)) {
                constexpr int s = decltype(s_tag)::value;
                const bf16x8 B = __builtin_bit_cast(bf16x8, rest[s]);
#pragma unroll
                for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[t][S::H + s], B, acc[t], 0, 0, 0);
                yy = square(rest[s], yy);
            });
            const float need = need_of(sum_of_halves(yy));
            if (passes(need)) {
                // which vectors pass: the masks of rows i (low half) and i + 4 (high half) of every register
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    unsigned long long m[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) m[i] = ballot64(acc[t][i] >= need);
                    if (lane == 0) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) *reinterpret_cast<unsigned long long*>(bits + it * 64 + t * 32 + 2 * i) = m[i];
                    }
                }
                met |= 1u << it;
            }
        }
    };
    next_records();
    for (int it = 0;; it += 3) {
        round(words_a, words_b, words_c, it);
        if (it + 1 >= n_it) break;
        round(words_b, words_c, words_a, it + 1);
        if (it + 2 >= n_it) break;
        round(words_c, words_a, words_b, it + 2);
        if (it + 3 >= n_it) break;
    }
    if (met == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // Lane = slot: its words (register 4 (r / 8) + r % 4 of block s / 32, half r / 4 % 2; r = s % 32), a place in its query's list
    // for all of them, then every lane writes its own.
    const int mine = (lane & 32) + 2 * (4 * ((lane >> 3) & 3) + (lane & 3)) + ((lane >> 2) & 1);
    uint32_t w[kFilterSteps], cnt = 0;
#pragma unroll
    for (int it = 0; it < kFilterSteps; ++it) {
        w[it] = ((met >> it) & 1u) && (uint32_t)lane < n_pairs ? bits[it * 64 + mine] : 0u;
        cnt += (uint32_t)__popc(w[it]);
    }
    if (cnt != 0) {
        const uint32_t base = atomicAdd(&a.counts[rec.x], cnt);
        const uint32_t seg0 = a.pairs[(size_t)rec.x * a.n_probes + 1].w, pos0 = a.pairs[(size_t)rec.x * a.n_probes + rec.y].w + item.v0;
        const size_t row = (size_t)rec.x * a.stride + seg0 + base;
        uint32_t* key = a.row_key + row;
        uint32_t* pos = a.row_pos + row;
#pragma unroll
        for (int it = 0; it < kFilterSteps; ++it)
            for (uint32_t left = w[it]; left != 0; left &= left - 1) {
                *key++ = rec.y;
                *pos++ = pos0 + (uint32_t)(it * 32) + (uint32_t)(__ffs((int)left) - 1);
            }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();          // the next item writes the words again
}

template <int BITS, int M, int STEPS>
__global__ void __launch_bounds__(kFilterThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
scan_filter_kernel(FilterArgs a) {
    using S = FilterShape<BITS, M, STEPS>;
    extern __shared__ __align__(16) unsigned char smem[];
    // LDS: codebooks in bf16 [sub-space][code][M] | per wave kWaveWords | ticket
    static_assert(S::book_bytes % 16 == 0, "the words behind the codebooks are aligned");
    uint32_t* const all_bits = reinterpret_cast<uint32_t*>(smem + S::book_bytes);
    uint32_t* const ticket = all_bits + kFilterWaves * kWaveWords;
    if (threadIdx.x == 0) *ticket = 0;
    for (int i = threadIdx.x; i < S::D * S::KSUB / 4; i += kFilterThreads) {
        const float4 x = reinterpret_cast<const float4*>(a.codebooks)[i];
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<bf16x4*>(smem + (size_t)i * 8) = bf16x4{(__bf16)x.x, (__bf16)x.y, (__bf16)x.z, (__bf16)x.w};
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    uint32_t* bits = all_bits + wave * kWaveWords;
    const uint32_t n_items = *a.n_items;
    // The items of a cluster are neighbours: a workgroup takes them eight at a time, so that the waves that read one cluster's
    // codes run on one compute unit.  (A counter of the whole grid evens out the ends but costs more: 2,048 waves that add to one
    // word at the start take 20 us.)
    auto take = [&]() {
        uint32_t t = 0;
        if (lane == 0) t = atomicAdd(ticket, 1u);
        t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
        return ((t >> 3) * gridDim.x + blockIdx.x) * 8u + (t & 7u);       // ascends with the ticket
    };
    auto record = [&](const Item& it) { return a.records[it.first + ((uint32_t)lane < it.n_pairs ? (uint32_t)lane : it.n_pairs - 1u)]; };
    uint32_t at = take();
    if (at >= n_items) return;
    Item item = item_of(a.items[2 * (size_t)at], a.items[2 * (size_t)at + 1]);
    uint4 rec = record(item);
    for (;;) {
        // the next item travels while this one is worked on: its description at once, its pairs from the second round on
        const uint32_t at_next = take();
        const bool more = at_next < n_items;
        const size_t where = 2 * (size_t)(more ? at_next : at);
        const uint4 d0 = a.items[where], d1 = a.items[where + 1];
        Item item_next;
        uint4 rec_next;
        auto next_records = [&]() __attribute__((always_inline)) {
            item_next = item_of(d0, d1);
            rec_next = record(item_next);
        };
        if (item.n_pairs > 32u) filter_item<BITS, M, STEPS, 2>(a, bits, item, rec, next_records);
        else filter_item<BITS, M, STEPS, 1>(a, bits, item, rec, next_records);
        if (!more) break;
        item = item_next;
        rec = rec_next;
        at = at_next;
    }
}

template <int BITS, int M, int STEPS>
int launch_shape(const FilterArgs& a, hipStream_t st) {
    using S = FilterShape<BITS, M, STEPS>;
    if constexpr (!S::valid) {
        return fail(IVFPQ_EUNSUPPORTED, "internal: no filter kernel for %d-bit codes of %d components", BITS, M);
    } else {
        auto kernel = scan_filter_kernel<BITS, M, STEPS>;
        if (int s = allow_full_lds(kernel)) return s;
        if (int s = require_no_static_lds(reinterpret_cast<const void*>(kernel))) return s;
        hipLaunchKernelGGL(kernel, dim3(256), dim3(kFilterThreads), filter_lds_bytes(BITS, S::D), st, a);
        HIP_TRY(hipGetLastError());
        return IVFPQ_OK;
    }
}
template <int BITS, int M>
int launch_dims(const FilterArgs& a, hipStream_t st) {
    switch (a.d) {
        case 64: return launch_shape<BITS, M, 4>(a, st);
        case 96: return launch_shape<BITS, M, 6>(a, st);
        case 128: return launch_shape<BITS, M, 8>(a, st);
        default: return fail(IVFPQ_EUNSUPPORTED, "internal: no filter kernel for %d components", a.d);
    }
}

}  // namespace

bool ivfpq::filter_supported(int bits, int pq_dim, int d, int chunk_width) {
    if (d != 64 && d != 96 && d != 128) return false;
    const int m = d / pq_dim;
    if (m * pq_dim != d || (m != 2 && !(m == 4 && (bits == 8 || bits == 4)))) return false;
    if (pq_dim * bits % 64 != 0) return false;
    const int cb = pq_dim * bits / 8;
    const int cw = (cb % 16 == 0 && cb / 16 <= 4 && (bits == 4 || bits == 8 || (bits == 6 && cb == 48))) ? 16 : 4;
    if (cw != chunk_width) return false;
    return filter_lds_bytes(bits, d) <= kLdsBytes && candidate_lds_bytes(bits, d) <= kLdsBytes;
}

size_t ivfpq::filter_lds_bytes(int bits, int d) { return ((size_t)d << bits) * 2 + (size_t)kFilterWaves * kWaveWords * 4 + 16; }

int ivfpq::launch_filter(const FilterArgs& a, hipStream_t st) {
    switch (a.bits * 8 + a.m) {
        case 8 * 8 + 2: return launch_dims<8, 2>(a, st);
        case 8 * 8 + 4: return launch_dims<8, 4>(a, st);
        case 7 * 8 + 2: return launch_dims<7, 2>(a, st);
        case 6 * 8 + 2: return launch_dims<6, 2>(a, st);
        case 5 * 8 + 2: return launch_dims<5, 2>(a, st);
        case 4 * 8 + 2: return launch_dims<4, 2>(a, st);
        case 4 * 8 + 4: return launch_dims<4, 4>(a, st);
        default: return fail(IVFPQ_EUNSUPPORTED, "internal: no filter kernel for %d-bit codes of %d components", a.bits, a.m);
    }
}
