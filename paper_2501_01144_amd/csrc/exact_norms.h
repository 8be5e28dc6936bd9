// Norms of rows, and whether they show that an output's fp32 sum is exact (gemm_native.hip, "Exact products").
#pragma once
#include "common.h"

namespace dfp4 {
namespace {

// Of the rows of a 32-row tile over a chunk of K, in units of the row (its reference: the smallest exponent of its
// nonzero blocks); every entry the largest over the rows, so that sums over chunks and maxima over tiles bound every row.
struct alignas(16) ExactStat {
    float sq;          // sum of squares
    float sq_low;      // sum of squares over blocks less than 4 binades above the reference
    float sum_high;    // sum of magnitudes over the other blocks
    float top;         // largest magnitude, at most
};

constexpr float kExactUnits = 16777216.0f * 0.9998f;  // the bounds' own rounding stays below 1e-4
// Rows whose reference lies outside these exponent bytes take the int32 path: a product of two units is then at least 2^-126
// (no partial sum is subnormal) and a sum of 2^24 of them below 2^127.
constexpr int kMinRef = 66, kMaxRef = 178;

// Whether sum |a||w| is at most 2^24 units for all of them: Cauchy-Schwarz over all blocks; or over the low blocks of one
// operand, and its high blocks (outlier channels) by their sum of magnitudes times the other's largest.  (Infinite norms and
// 0 times infinity fail every comparison.)
__device__ __forceinline__ bool sums_exactly(const ExactStat& a, const ExactStat& w) {
    return sqrtf(a.sq) * sqrtf(w.sq) <= kExactUnits || sqrtf(a.sq_low) * sqrtf(w.sq) + a.sum_high * w.top <= kExactUnits ||
           sqrtf(a.sq) * sqrtf(w.sq_low) + a.top * w.sum_high <= kExactUnits;
}

}  // namespace
}  // namespace dfp4
