// Adjust-Bin-Bounds of one axis by one workgroup, for the steps kernels and the
// batch (see steps.hip for what its sums share with the host's steps).
#pragma once

#include "estimate_device.hpp"
#include "internal.hpp"

namespace mcubes {

constexpr int kRefineThreads = 256;

// The workgroup's threads each take a contiguous run of [first, last): the
// run of thread t.
__device__ __forceinline__ void thread_run(int first, int last, int *a, int *b) {
    const int per = (last - first + (int)blockDim.x - 1) / (int)blockDim.x;
    *a = min(first + (int)threadIdx.x * per, last);
    *b = min(*a + per, last);
}

// x[0] + ... + x[n-1] in a fixed order: each thread its run in order, then a
// butterfly across the wave (every lane ends with the same value), then the
// waves in order.  Returned to every thread.
__device__ inline double block_sum(const double *x, int n, double *wave_tmp) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int a, b;
    thread_run(0, n, &a, &b);
    double s = 0.0;
    for (int i = a; i < b; ++i) s = s + x[i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s = s + __shfl_xor(s, off, 64);
    if (lane == 0) wave_tmp[wave] = s;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < nw; ++w) t = t + wave_tmp[w];
    __syncthreads();
    return t;
}

// In place over [first, last): E[k] = max(lo, E[first], ..., E[k]).  Each
// thread its run, the runs' maxima scanned across the wave and the waves.
// Max is exact, so the grouping does not change the result.
__device__ inline void running_max(double *E, int first, int last, double lo, double *wave_tmp) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int a, b;
    thread_run(first, last, &a, &b);
    double m = lo;
    for (int k = a; k < b; ++k) m = fmax(E[k], m);
    double x = m;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double y = __shfl_up(x, off, 64);
        if (lane >= off) x = fmax(x, y);
    }
    if (lane == 63) wave_tmp[wave] = x;
    __syncthreads();
    double before = lo;
    for (int w = 0; w < wave; ++w) before = fmax(before, wave_tmp[w]);
    const double left = __shfl_up(x, 1, 64);
    if (lane > 0) before = fmax(before, left);
    double run = before;
    for (int k = a; k < b; ++k) {
        run = fmax(E[k], run);
        E[k] = run;
    }
    __syncthreads();
}

// Running sums P[0] = 0, P[i + 1] = x[0] + ... + x[i]: each thread its run
// in order, after the total of everything before it (the runs' totals
// scanned across the wave, then the waves in order).  The rounding of the
// cross-run sums can leave a later P an ulp below an earlier one, so P is
// then made non-decreasing (a running maximum, exact).
__device__ inline void running_sums(const double *x, int n, double *P, double *wave_tmp) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int a, b;
    thread_run(0, n, &a, &b);
    double s = 0.0;
    for (int i = a; i < b; ++i) s = s + x[i];
    double incl = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double y = __shfl_up(incl, off, 64);
        if (lane >= off) incl = incl + y;
    }
    if (lane == 63) wave_tmp[wave] = incl;
    __syncthreads();
    double before = 0.0;
    for (int w = 0; w < wave; ++w) before = before + wave_tmp[w];
    const double left = __shfl_up(incl, 1, 64);
    if (lane > 0) before = before + left;
    double run = before;
    for (int i = a; i < b; ++i) {
        run = run + x[i];
        P[i + 1] = run;
    }
    if (threadIdx.x == 0) P[0] = 0.0;
    __syncthreads();
    running_max(P, 1, n + 1, 0.0, wave_tmp);
}

// Adjust-Bin-Bounds of one axis by one workgroup of kRefineThreads.  On entry
// C (nb doubles, in LDS or device memory) holds the axis's contributions and
// the LDS arrays follow lds: the compressed weights r (nb), their running
// sums P (nb + 1), the old boundaries (nb + 1) and the new ones E (nb + 1).
// C may be E itself: it is read before E is written.  Returns the new
// boundaries, in LDS: E, or the old ones where the axis has no usable weight.
// ROOT32: see compressed_share.  Ends with a workgroup barrier.
template <bool ROOT32>
__device__ __forceinline__ const double *adjusted_axis(double *lds, const double *C, const double *B, int nb,
                                                       double alpha) {
    double *r = lds, *P = r + nb, *prev = P + nb + 1, *E = prev + nb + 1;
    __shared__ double wave_tmp[kRefineThreads / 64];
    const int tid = threadIdx.x;
    for (int i = tid; i <= nb; i += kRefineThreads) prev[i] = B[i];
    // three-point smoothing (two points at the ends)
    for (int i = tid; i < nb; i += kRefineThreads) {
        double s;
        if (i == 0) s = (C[0] + C[1]) / 2.0;
        else if (i == nb - 1) s = (C[nb - 2] + C[nb - 1]) / 2.0;
        else s = ((C[i - 1] + C[i]) + C[i + 1]) / 3.0;
        r[i] = s;
    }
    __syncthreads();
    const double S = block_sum(r, nb, wave_tmp);
    bool moved = S > 0.0 && isfinite(S);  // else the axis keeps its boundaries
    if (moved) {
        // Lepage's damped compression of each bin's share
        for (int i = tid; i < nb; i += kRefineThreads) r[i] = compressed_share<ROOT32>(r[i], S, alpha);
        __syncthreads();
        running_sums(r, nb, P, wave_tmp);
        moved = P[nb] > 0.0;
    }
    if (moved) {
        // boundary k closes k equal shares of the compressed weight: the
        // host's scan stops at the first bin s with s = nb - 1 or
        // P[s + 1] >= goal (P is non-decreasing, so that test is monotone in
        // s) and interpolates inside it
        const double per_bin = P[nb] / (double)nb;
        for (int k = 1 + tid; k < nb; k += kRefineThreads) {
            const double goal = (double)k * per_bin;
            int lo = 0, hi = nb - 1;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (P[mid + 1] < goal) lo = mid + 1;
                else hi = mid;
            }
            const int src = lo;
            double frac = r[src] > 0.0 ? (goal - P[src]) / r[src] : 0.0;
            frac = fmin(fmax(frac, 0.0), 1.0);
            E[k] = __fma_rn(frac, prev[src + 1] - prev[src], prev[src]);
        }
        __syncthreads();
        // boundaries never decrease: each is at least the one before (the
        // first at least the old lower end)
        running_max(E, 1, nb, prev[0], wave_tmp);
        if (tid == 0) {
            E[0] = 0.0;
            E[nb] = 1.0;
        }
        __syncthreads();
    }
    return moved ? E : prev;
}

}  // namespace mcubes
