// How a pass of a table larger than the LDS is summed in FP32, and the error
// of that sum.  (Plain C++ but for the execution-space names.)
#pragma once

#include <stdint.h>

namespace bns {

// A stratum per lane (strata_partial) where a pass has strata for half of its
// lanes at least: with few strata of many cells most lanes would idle and one
// would add hundreds of terms (X of 5 and Y of 200 categories: 5 strata of
// 1,000 cells a pass, of 256 lanes), and its cells go to all lanes
// (stat_partial): 180 tests of depth 2 of such variables, 100,000 samples, X^2,
// 942 us by strata and 353 by cells; passes of hundreds of strata the same as
// by strata alone (220 x 100,000, depths 5 and 6).
__host__ __device__ inline bool strata_by_lane(uint32_t rx, uint32_t zc_per, uint32_t lanes) {
    return rx >= 2u && rx <= 5u && 2u * zc_per >= lanes;
}

// Terms one lane adds in a pass at most.
__host__ __device__ inline double lane_terms(uint32_t rxy, uint32_t zc_per, uint32_t lanes, bool by_lane) {
    return by_lane ? (double)(rxy * ((zc_per + lanes - 1u) / lanes)) : (double)(rxy * zc_per) / (double)lanes + 1.0;
}

// Relative error bound of the FP32 G^2 sum: every summand is non-negative and
// carries at most a few tens of ulp of error (conversions, reciprocals, the
// series or the log2), and each lane adds up to lane_terms of them before a
// tree, so the relative error stays below (32 + terms) * 2^-24 per pass.
__host__ __device__ inline double fp32_sum_bound(double terms, uint32_t passes) {
    return (32.0 + terms) * 5.96e-8 * (double)passes + 1e-6;
}

}  // namespace bns
