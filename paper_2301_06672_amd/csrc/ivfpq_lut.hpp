// Table entries: the conversions between FP32 and the storage types of a lookup table (fp32, half, e5m3, e4m4), and
// the direct-form distance of one entry.  Included by .hip translation units only; the code has internal linkage.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include "ivfpq_internal.hpp"

namespace ivfpq {

struct Fp8Params { int lo, hi, sub; };   // of fp8_params below

// Encoding of an 8-bit table as the caller configured it: fixed constants, or a bias chosen per table.
struct Fp8Mode {
    Fp8Params fixed;     // constants for the configured bias and rounding
    int truncate;        // rounding of the encode: 0 nearest (ties up), 1 truncate
    int per_table;       // 1: the bias follows the largest entry of each table
};

}  // namespace ivfpq

namespace {

using ivfpq::Fp8Mode;
using ivfpq::Fp8Params;

template <int LUT> struct LutTraits;     // bytes: size of one table entry
template <> struct LutTraits<IVFPQ_LUT_FP32> { static constexpr int bytes = 4; };
template <> struct LutTraits<IVFPQ_LUT_FP16> { static constexpr int bytes = 2; };
template <> struct LutTraits<IVFPQ_LUT_FP8_E5M3> { static constexpr int bytes = 1; };
template <> struct LutTraits<IVFPQ_LUT_FP8_E4M4> { static constexpr int bytes = 1; };
// The two 8-bit formats.  shift: how far a code is shifted to line up with the FP32 exponent/mantissa
// field (23 less the mantissa bits); top_exp: the largest exponent field; bias_min/bias_max: range of
// the exponent bias for which every code is a finite normal FP32 number.
template <int LUT> struct Fp8Format {     // e5m3
    static constexpr int shift = 20, top_exp = 31, bias_min = -96, bias_max = 110;
};
template <> struct Fp8Format<IVFPQ_LUT_FP8_E4M4> {
    static constexpr int shift = 19, top_exp = 15, bias_min = -100, bias_max = 110;
};
template <int LUT> constexpr bool kIsFp8 = LUT == IVFPQ_LUT_FP8_E5M3 || LUT == IVFPQ_LUT_FP8_E4M4;

// Constants of a sign-less 8-bit float (Sec. II) with M mantissa bits (shift = 23 - M) and exponent
// bias B: value(b) = (1 + mant/2^M) * 2^(exp - B).  Both conversions are a shift plus a bias
// adjustment on the FP32 bit pattern:
//   code = (clamp_s32(bits, lo, hi) - sub) >> shift        bits = (code << shift) + lo
// lo = (127 - B) << 23 is the smallest value, hi = lo + (255 << shift) the largest; sub = lo less half
// an 8-bit ulp, so that the shift rounds to nearest with ties up, or lo itself to truncate.  The clamp
// acts on the pattern as a signed integer: zero and negatives give code 0, +Inf code 255.
// e5m3 with B = 15: lo = 0x38000000, hi = 0x47F00000, sub = 0x37F80000.
__host__ __device__ inline Fp8Params fp8_params(int shift, int bias, int truncate) {
    Fp8Params p;
    p.lo = (127 - bias) << 23;
    p.hi = p.lo + (255 << shift);
    p.sub = truncate ? p.lo : p.lo - (1 << (shift - 1));
    return p;
}
// The code of x, left in the TOP byte of the result (low bits undefined): the clamp is one
// three-operand median once the upper limit sits in a vector register (`hi_v`; an instruction takes
// one scalar operand only), the bias subtraction and the shift are one add-shift.
template <int SHIFT>
__device__ inline uint32_t fp8_code_top_byte(float x, const Fp8Params p, int hi_v) {
    int b;
    uint32_t t;
    const int nsub = -p.sub;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(b) : "v"(__float_as_int(x)), "s"(p.lo), "v"(hi_v));     // clamp to [lo, hi]
    asm("v_add_lshl_u32 %0, %1, %2, %3" : "=v"(t) : "v"(b), "s"(nsub), "n"(24 - SHIFT));            // (b - sub) << (24 - SHIFT)
    return t;
}
// four codes (of f[0..3], lowest byte first) gathered from the top bytes with three byte permutes
template <int SHIFT>
__device__ inline uint32_t fp8_pack4(const float f[4], const Fp8Params p, int hi_v) {
    const uint32_t t0 = fp8_code_top_byte<SHIFT>(f[0], p, hi_v), t1 = fp8_code_top_byte<SHIFT>(f[1], p, hi_v);
    const uint32_t t2 = fp8_code_top_byte<SHIFT>(f[2], p, hi_v), t3 = fp8_code_top_byte<SHIFT>(f[3], p, hi_v);
    // selector bytes: 0-3 pick a byte of the second operand, 4-7 of the first, 0x0c gives zero
    const uint32_t p01 = __builtin_amdgcn_perm(t1, t0, 0x0c0c0703u);
    const uint32_t p23 = __builtin_amdgcn_perm(t3, t2, 0x07030c0cu);
    return p01 | p23;
}
template <int SHIFT>
__device__ inline float fp8_to_f32(uint32_t b, const Fp8Params p) { return __uint_as_float((b << SHIFT) + (uint32_t)p.lo); }

// IEEE half, round to nearest even, saturating at the largest finite half.
__device__ inline uint32_t half_bits_from_f32(float x) {
    float c = x > 65504.0f ? 65504.0f : x;
    return (uint32_t)__half_as_ushort(__float2half_rn(c));
}

// One table entry: sum over the sub-vector, left to right, of (cb - rq)^2 with one rounding per
// step (subtract, then fused multiply-add into the running sum).
template <int M>
__device__ inline float lut_entry(const float* cbv, const float* rq) {
    float acc = 0.f;
#pragma unroll
    for (int t = 0; t < M; ++t) {
        float diff = cbv[t] - rq[t];
        acc = __builtin_fmaf(diff, diff, acc);
    }
    return acc;
}
}  // namespace
