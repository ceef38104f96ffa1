// The numbers of the matrix-core filter's bound: by how much a stored sum, a bf16 product and a few fp32 roundings can miss the
// squared distance they stand for.  Plain C++, so that a test can take the same numbers.
#pragma once

#include <cmath>

#include "../../include/ivfpq.h"

namespace ivfpq {

constexpr float kSquareLoss = 0.00394f;        // a sum of squares of bf16 roundings is at most 1 + this times the sum of the squares
constexpr float kRoundedNorm = 1.008f;         // ... and a squared norm at most this times that of its bf16 rounding
constexpr float kEntrySlack = 1.00001f;        // roundings of an entry's largest value, (|r_j| + largest codeword)^2
constexpr float kHiddenSlack = 1.0001f;        // roundings of the sum of what saturation can hide
constexpr float kLimitShare = 0.0625f;         // share of eta by which the limit itself is widened
constexpr float kWordNormSlack = 1.0001f;      // roundings of the largest codeword's norm
// of norms that are compared to leave out a whole cluster: a relative 2^-13 for the rounding of either, sums of at most 128 squares
constexpr float kCullNear = 0.99987f, kCullRadius = 1.00013f, kCullLimit = 1.0001f, kCullTop = 0.9999f;

// The largest share of an entry that its stored form is below it: half 2^-11, 8-bit formats of M mantissa bits 1 / (2^(M+1) + 1) rounded to
// nearest, 1 / (2^M + 1) truncated.
inline double stored_loss(int lut_dtype, bool truncate) {
    if (lut_dtype == IVFPQ_LUT_FP32) return 0.0;
    if (lut_dtype == IVFPQ_LUT_FP16) return 1.0 / 2048;
    const int mantissa = lut_dtype == IVFPQ_LUT_FP8_E5M3 ? 3 : 4;
    return 1.0 / ((1 << (truncate ? mantissa : mantissa + 1)) + 1);
}

// What |r - y|^2 of a vector with R <= bound is limited by: bound * scale + add, where no entry saturates (the kernel sees to
// those that may).  A stored entry is below its distance by at most the share stored_loss (and 2^-25 where a half is subnormal); the 2^-15 cover the
// sum of up to 128 entries and the rounding of an entry's own distance.  eta: r.y is formed from bf16 operands (2^-8 + 2^-18 of the sum
// of magnitudes, which is at most (|r|^2 + |y|^2) / 2), summed with the threshold in any order (4 (d + 2) 2^-24 of either, with
// a factor 4 of slack as for the ranking values), |r|^2 is a sum of d squares.
struct FilterBound {
    float scale, add, eta;
};
inline FilterBound filter_bound(int lut_dtype, bool truncate, int pq_dim, int d) {
    const double loss = stored_loss(lut_dtype, truncate), below = lut_dtype == IVFPQ_LUT_FP16 ? pq_dim * std::ldexp(1.0, -25) : 0.0;
    return FilterBound{(float)((1.0 + std::ldexp(1.0, -15)) / (1.0 - loss)), (float)(below / (1.0 - loss) * 1.001 + 1e-30),
                       (float)(0.00392 + (12.0 * d + 64.0) * std::ldexp(1.0, -24))};
}

}  // namespace ivfpq
