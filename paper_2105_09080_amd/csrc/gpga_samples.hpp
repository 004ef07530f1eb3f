// Pieces shared by the kernels on stored and regenerated features: lane reductions and the terms of a sample.
#pragma once

#include "gpga_internal.hpp"

// Lane-shift reductions on the data-parallel-primitive path of the vector ALU (no LDS
// round trips): a 64-bit value moved as two 32-bit halves from the lane CTRL selects.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u & 0xffffffffull), CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double readlane_f64(double v, int src_lane) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u & 0xffffffffull), src_lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), src_lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Sum over each aligned row of 16 lanes (shifts by 1, 2, 4, 8 within the row; a lane without
// a source adds 0); complete in the row's last lane.  Every lane of the wavefront must be active.
__device__ __forceinline__ double row16_sum_last(double v) {
    v += dpp_f64<0x111>(v);  // row_shr:1
    v += dpp_f64<0x112>(v);  // row_shr:2
    v += dpp_f64<0x114>(v);  // row_shr:4
    v += dpp_f64<0x118>(v);  // row_shr:8
    return v;
}
// Halves (rows of 16 otherwise) exchanged between two values and added: with halves, lanes 0 to 31 hold a[l] + a[l + 32] and
// the others b[l - 32] + b[l]; without, rows 0 and 2 the sums of a's rows 0, 1 and 2, 3, rows 1 and 3 those of b's.
__device__ __forceinline__ double swap_add(double a, double b, bool halves) {
    const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
    uint32_t a0 = (uint32_t)ua, a1 = (uint32_t)(ua >> 32), b0 = (uint32_t)ub, b1 = (uint32_t)(ub >> 32);
    if (halves) {
        const auto lo = __builtin_amdgcn_permlane32_swap(a0, b0, false, false), hi = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
        a0 = lo[0], b0 = lo[1], a1 = hi[0], b1 = hi[1];
    } else {
        const auto lo = __builtin_amdgcn_permlane16_swap(a0, b0, false, false), hi = __builtin_amdgcn_permlane16_swap(a1, b1, false, false);
        a0 = lo[0], b0 = lo[1], a1 = hi[0], b1 = hi[1];
    }
    return __longlong_as_double((long long)(((uint64_t)a1 << 32) | a0)) + __longlong_as_double((long long)(((uint64_t)b1 << 32) | b0));
}
// Per-sample coefficient and loss term from the margin z.
//   least squares: r = z - b          coef = r / B           loss = r^2 / (2B)
//   logistic     : t = y z            coef = -y s(-t) / B    loss = ln(1 + e^{-t}) / B
template <int KIND>
__device__ __forceinline__ float sample_coefficient(double z, float target, float invB) {
    if (KIND == PROB_LSQ) return (float)((z - (double)target) * invB);
    const double t = (double)target * z;
    const double e = exp(-fabs(t));                                    // in (0,1], never overflows
    const double sig = (t >= 0.0 ? e : 1.0) / (1.0 + e);               // sigma(-t)
    return (float)(-(double)target * sig * invB);
}
template <int KIND>
__device__ __forceinline__ float sample_loss(double z, float target, float invB) {
    if (KIND == PROB_LSQ) {
        const double r = z - (double)target;
        return (float)(0.5 * r * r * invB);
    }
    const double t = (double)target * z;
    return (float)((fmax(-t, 0.0) + log1p(exp(-fabs(t)))) * invB);
}
template <int KIND>
__device__ __forceinline__ void sample_terms(double z, float target, float invB, float* coef, float* loss) {
    *coef = sample_coefficient<KIND>(z, target, invB);
    *loss = sample_loss<KIND>(z, target, invB);
}
