// Soft regime: the quantizer's quantities from a table (cdl_soft.hip; not installed).
#pragma once

#include "cdl_finish.h"
#include "cdl_marginal.h"
#include "cdl_quantizer_math.h"

namespace cdl {

// (kSoftMaxBins, kSoftTableBytes, kSoftFrom: cdl_internal.h)
// moments of an interval; one more where the intervals are fine, and their number so that the rows of the blocks hold them
constexpr int kSoftMoments = 6, kSoftMoreMoments = 7;
constexpr int kSoftMoreBins = kSoftMoments * kSoftMaxBins / kSoftMoreMoments;
constexpr int kSoftThreads = 1024;
constexpr int kSoftRowWords = kSoftMoments * kSoftMaxBins + 256;

// Workspace of the forward pass: the table, then the rows of the blocks' moments.
int64_t soft_fwd_grid(int64_t n);
size_t soft_fwd_bytes(int64_t n, int32_t n_levels);

struct SoftPlan {
    int bins;              // 0: another kernel serves
    int fine;              // sets that the kernels in double serve otherwise: intervals of sigma / 8, else sigma / 4
    int small_set;         // at most 33 levels: entries outside the table's range in double, as the kernels for them do
    double half_range;     // the table covers |r| <= half_range, r = theta / delta - c0
    double inv_h;          // bins per unit of r
    double c0, inv_delta, delta;
    double kappa;
};

// Whether the table serves (soft regime, full CPMF, a tensor large enough).
SoftPlan soft_plan(const cdl_qparams &p, const QConst &k, int64_t n, bool fine);

int launch_soft_fwd(const float *theta, int64_t n, const cdl_qparams &p, const QConst &k, const SoftPlan &s, int8_t *idx, float *soft,
                    const MargFinish &fin, void *ws, hipStream_t stream);
int launch_soft_bwd(const float *theta, const float *g, int64_t n, const cdl_qparams &p, const QConst &k, const SoftPlan &s, float *dtheta,
                    const ScalarFinish &fin, void *table, int grid, hipStream_t stream);

}  // namespace cdl
