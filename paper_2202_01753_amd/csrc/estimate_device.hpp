// Weighted-Estimates by one wavefront, and the compression of Adjust-Bin-Bounds,
// for the kernels that run the steps of Alg. 2 on the device.
#pragma once

#include "estimate.hpp"

namespace mcubes {

// The value of lane i (the same i for every lane) of a wavefront.
__device__ __forceinline__ double lane_value(double x, int i) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), i),
                            __builtin_amdgcn_readlane(__double2loint(x), i));
}

// weighted_estimate by one wavefront, for k <= 64: lane i holds I_i and var_i.
// The divisions are the lanes' own, the sums are formed in the same order as
// there, so the result is the same bit for bit; every lane gets it.  (One
// lane reading the passes one after the other from memory took 5 us for ten.)
__device__ inline void wave_weighted_estimate(int k, double I, double var, double *out) {
    const bool in = (int)(threadIdx.x & 63) < k;
    const uint64_t zero_var = __ballot(in && var == 0.0), no_info = __ballot(in && var == 0.0 && I == 0.0);
    const uint64_t all = k >= 64 ? ~0ull : (1ull << k) - 1;
    const int used = __popcll(all & ~no_info);
    uint64_t exact = zero_var & ~no_info;
    if (used == 0) {
        out[0] = 0.0;
        out[1] = INFINITY;
        out[2] = NAN;
        return;
    }
    if (exact) {
        const int n = __popcll(exact);
        double sum = 0.0;
        for (; exact; exact &= exact - 1) sum = sum + lane_value(I, __ffsll((unsigned long long)exact) - 1);
        out[0] = sum / (double)n;
        out[1] = 0.0;
        out[2] = used > 1 ? 0.0 : NAN;
        return;
    }
    const uint64_t weighted = all & ~zero_var;
    const double w = 1.0 / var, wi = w * I;
    double wsum = 0.0, wisum = 0.0;
    for (uint64_t m = weighted; m; m &= m - 1) {
        const int i = __ffsll((unsigned long long)m) - 1;
        wsum = wsum + lane_value(w, i);
        wisum = wisum + lane_value(wi, i);
    }
    const double mean = wisum / wsum;
    const double dv = I - mean, q = (dv * dv) / var;
    double chi = 0.0;
    for (uint64_t m = weighted; m; m &= m - 1) chi = chi + lane_value(q, __ffsll((unsigned long long)m) - 1);
    out[0] = mean;
    out[1] = 1.0 / sqrt(wsum);
    out[2] = used > 1 ? chi / (double)(used - 1) : NAN;
}

// Lepage's damped compression of a bin's share s of the axis total S (0 < S
// finite): ((1 - s/S) / ln(S/s))^alpha, 0 for s = 0 and 1 for s = S.  ROOT32: the
// usual exponent 3/2 as q sqrt(q), two correctly rounded operations (a relative
// error of at most 2^-52) at a tenth of the power function's instructions
// (where many bins share few threads: fused and batched adjustment).  Boundaries
// against extended precision on 60 histograms of 100 to 500 bins, root mean square:
// 1.1e-16 with either in adjusted_axis's order of sums, 6.9e-16 with either in the
// host's, one bin after another.
template <bool ROOT32>
__device__ __forceinline__ double compressed_share(double s, double S, double alpha) {
    if (s == 0.0) return 0.0;
    if (s == S) return 1.0;
    const double q = (1.0 - s / S) / log(S / s);
    return ROOT32 && alpha == 1.5 ? q * sqrt(q) : pow(q, alpha);
}

}  // namespace mcubes
