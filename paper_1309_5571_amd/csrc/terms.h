// Diagonal terms of an output element (device), shared by the projection kernels.
#pragma once

#include "internal.h"
#include "lanes.h"

namespace dmrg {

// diagonal-term contribution at output element (rr, cc) of a task's pair
__device__ __forceinline__ double diag_sum(const DiagTerm *__restrict__ diags, int d0, int d1,
                                           const double *__restrict__ coef, double x, int64_t rr, int64_t cc) {
    double val = 0.0;
    for (int d = d0; d < d1; ++d) {
        const DiagTerm dt = diags[d];
        double w = (coef ? coef[dt.coef] : 1.0) * dt.w * x;
        if (dt.vl) w *= as_global(dt.vl)[rr * dt.sl];
        if (dt.vr) w *= as_global(dt.vr)[cc * dt.sr];
        val += w;
    }
    return val;
}

}  // namespace dmrg
