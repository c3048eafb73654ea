// The device-side plan of a backward call: scale of the gradient and limb counts (not installed).
#pragma once

#include "cdl_internal.h"

#include <math.h>

namespace cdl {

constexpr int kMinLimbs = 3, kMaxLimbs = 6;

struct BwdPlan {
    int limbs_da, limbs_db;          // limbs used for d_a_hat / d_b_hat
    float gscale_da, gscale_db;      // 2^(8L-1) / sigma
    double out_scale_da, out_scale_db;  // delta_b * sigma / 2^(8L-1), delta_a * sigma / 2^(8L-1)
    double bound_da, bound_db;          // what the rounding of g can change in one entry of d_a_hat / d_b_hat, at most
};

// Chooses the power-of-two scale of g and, for each backward product, the number of limbs.  With
// sigma = 2^e > 1.01 max|g| and L limbs, q = rint(g 2^(8L-1)/sigma) is off by at most half a unit, i.e. every
// entry of g is represented to within sigma 2^-8L, so one output of a product, delta * sum_c g_c idx_c, is off by
// at most delta sigma 2^-8L sum_c |idx_c| whatever the signs and values of g: a bound, not an estimate.  The
// largest sum of |idx| over the contraction (one per output column: col_abs_a / col_abs_b, from whoever reads the operands first)
// goes in, and L is the smallest count (3..6) that brings the bound under 9e-7 - the absolute part of the
// parity tolerance, less a margin for the roundings of the recombination and of the fp32 result, which are
// relative (1e-7) and covered by its relative part.  If six limbs do not reach it (contractions of many
// millions of large indices) six are used and the bound, stored in the plan, says what was reached.
constexpr double kLimbBoundTarget = 9e-7;

// The diagnostic words of a call whose products were formed directly (one thread): no limbs, nothing rounded.
__device__ __forceinline__ void no_limbs(BwdPlan *plan)
{
    plan->limbs_da = plan->limbs_db = 0;
    plan->bound_da = plan->bound_db = 0.0;
}

// (one thread; amax_bits: the largest |g| as the bits of a float)
__device__ __forceinline__ void choose_limbs(BwdPlan *plan, unsigned int amax_bits, unsigned int col_abs_a, unsigned int col_abs_b,
                                             float delta_a, float delta_b)
{
    const float amax = __uint_as_float(amax_bits);
    int e = 0;
    if (amax > 0.0f) frexpf(amax * 1.01f, &e);   // amax * 1.01 = f 2^e with f in [0.5, 1)
    e = max(min(e, 127), -80);                   // keeps 2^(8L-1-e) a normal float for every L
    // d_a_hat contracts g with b_idx (step delta_b), d_b_hat with a_idx (step delta_a)
    const double unit_da = (double)delta_b * (double)col_abs_b, unit_db = (double)delta_a * (double)col_abs_a;
    int la = kMinLimbs, lb = kMinLimbs;
    while (la < kMaxLimbs && unit_da * ldexp(1.0, e - 8 * la) > kLimbBoundTarget) ++la;
    while (lb < kMaxLimbs && unit_db * ldexp(1.0, e - 8 * lb) > kLimbBoundTarget) ++lb;
    plan->bound_da = unit_da * ldexp(1.0, e - 8 * la);
    plan->bound_db = unit_db * ldexp(1.0, e - 8 * lb);
    plan->limbs_da = la;
    plan->limbs_db = lb;
    plan->gscale_da = ldexpf(1.0f, 8 * la - 1 - e);
    plan->gscale_db = ldexpf(1.0f, 8 * lb - 1 - e);
    plan->out_scale_da = (double)delta_b * ldexp(1.0, e + 1 - 8 * la);
    plan->out_scale_db = (double)delta_a * ldexp(1.0, e + 1 - 8 * lb);
}

}  // namespace cdl
