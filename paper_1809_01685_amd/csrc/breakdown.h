// The breakdown test of the Lanczos recurrence.
#pragma once
#include "wave.h"

namespace tnslq {
namespace {

constexpr double BREAKDOWN_TOL = 1e-12;

// Step (1-based) at which the probe broke down among steps 1..jmax, or 0.
// Breakdown at step s: beta_{s+1} <= tol * (max_{i<=s} |alpha_i| + max_{2<=i<=s} beta_i).
// Called by whole waves: lane i tests step i + 1 against running maxima taken
// by a scan over the lanes (one thread walking the steps waited for memory at
// each one, 5 us in each pass at step 40).  amax and bmax: the maxima over
// all jmax steps.
__device__ inline int first_break(const double *alpha_k, const double *beta_k, int jmax, double &amax, double &bmax) {
    const int lane = threadIdx.x & 63;
    amax = bmax = 0.0;
    for (int s0 = 0; s0 < jmax; s0 += 64) {
        const int s = s0 + lane + 1;
        const bool in = s <= jmax;
        double a = in ? fabs(alpha_k[s - 1]) : 0.0, b = in && s >= 2 ? beta_k[s - 1] : 0.0;
        const double next = in ? beta_k[s] : INFINITY;
        a = fmax(a, amax);
        b = fmax(b, bmax);
        a = wave_scan_max(a);
        b = wave_scan_max(b);
        const unsigned long long hit = __ballot(in && next <= BREAKDOWN_TOL * (a + b));
        if (hit) return s0 + __builtin_ctzll(hit) + 1;
        amax = lane_value(a, 63);
        bmax = lane_value(b, 63);
    }
    return 0;
}
__device__ inline int first_break(const double *alpha_k, const double *beta_k, int jmax) {
    double amax, bmax;
    return first_break(alpha_k, beta_k, jmax, amax, bmax);
}

}  // namespace
}  // namespace tnslq
