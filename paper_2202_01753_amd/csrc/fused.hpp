// The steps of Alg. 2 between two passes inside the sampling launch of the
// second (fused runs, see FusedArgs): the merge of the previous pass's
// totals, Weighted-Estimates and Check-Convergence, and Adjust-Bin-Bounds, by
// every workgroup for itself.
//
// Bound: latency, a chain of one trip to memory, seven barriers and the log of a
// bin or two per thread.  The same steps in a launch of their own
// (steps_kernel) cost that chain, two more trips to memory, one to the host
// mirror and the gap between two dependent launches (figures at
// kFusedMaxBins).
#pragma once

#include "estimate_device.hpp"
#include "internal.hpp"

namespace mcubes {
namespace fused {

__device__ __forceinline__ void two_sum_merge(double &s, double &c, double s2, double c2) {
    const double t = s + s2;
    const double bp = t - s;
    const double e = (s - (t - bp)) + (s2 - bp);
    s = t;
    c = (c + c2) + e;
}

// Lane's share of [first, last): a contiguous run, the wave's runs in lane order.
__device__ __forceinline__ void lane_run(int first, int last, int lane, int *a, int *b) {
    const int per = (last - first + 63) >> 6;
    *a = min(first + lane * per, last);
    *b = min(*a + per, last);
}

// The row of flat index e in rows of nb, for e below 2^16: the float quotient
// of e + 1/2 is at least 1/(2 nb) away from every integer, its error below
// 1e-5.
__device__ __forceinline__ int row_of(int e, float inv_nb) { return (int)(((float)e + 0.5f) * inv_nb); }

// In place over x[first..last): x[k] = max(lo, x[first], ..., x[k]), by one wave.
__device__ __forceinline__ void wave_running_max(double *x, int first, int last, double lo, int lane) {
    int a, b;
    lane_run(first, last, lane, &a, &b);
    double m = lo;
    for (int k = a; k < b; ++k) m = fmax(x[k], m);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double y = __shfl_up(m, off, 64);
        if (lane >= off) m = fmax(m, y);
    }
    const double left = __shfl_up(m, 1, 64);
    double run = lane > 0 ? left : lo;
    for (int k = a; k < b; ++k) {
        run = fmax(x[k], run);
        x[k] = run;
    }
}

// The workgroup is through with the pass that ended the run: the last one to
// say so clears the accumulators and the flag that the others still read.
__device__ __forceinline__ void leave(const SampleArgs &a, int32_t *last_wg) {
    const FusedArgs &z = a.fused;
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        *last_wg = atomicAdd(&z.state->ticket, 1u) == gridDim.x - 1 ? 1 : 0;
    }
    __syncthreads();
    if (!*last_wg) return;
    __threadfence();
    for (int i = threadIdx.x; i < kFusedAccs * a.hist_stride; i += blockDim.x) z.prev_acc[i] = 0.0;
    if (threadIdx.x == 0) {
        *z.prev_flag = 0u;
        z.state->ticket = 0u;
    }
}

// Everything before pass a.iter; returns true if the run has ended.  On
// return (false) *bounds holds the pass's boundaries, D rows of nb + 1, in the
// scratch LDS (fused_scratch doubles).  Ends with a workgroup barrier.
template <int D>
__device__ __forceinline__ bool steps(const SampleArgs &a, double *scratch, const double **bounds) {
    const FusedArgs &z = a.fused;
    __shared__ double axis_sum[D];
    __shared__ double est_s[3];
    __shared__ int32_t status_s, last_wg;
    const int nb = a.nb, row = nb + 1, total = D * row;
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = tid >> 6, waves = nthr >> 6;
    const bool first_wg = blockIdx.x == 0;
    const float inv_nb = 1.0f / (float)nb, inv_row = 1.0f / (float)row;
    double *E = scratch, *C = E, *r = E + total, *P = r + total, *prev = P + total;

    // the next pass's accumulators and flag
    auto clear_next = [&]() {
        for (int i = blockIdx.x * nthr + tid; i < kFusedAccs * a.hist_stride; i += gridDim.x * nthr) z.clear_acc[i] = 0.0;
        if (first_wg && tid == 0) *z.clear_flag = 0u;
    };
    if (z.prev_blocks == 0) {  // the first pass: Init-Bins and the run's state
        clear_next();  // (the sets of passes 1 and 2 hold anything when a run starts)
        for (int e = tid; e < total; e += nthr) {
            const double b = (double)(e - row * row_of(e, inv_row)) / (double)nb;
            E[e] = b;
            if (first_wg) z.next_grid[e] = b;
        }
        if (first_wg && tid == 0) {
            RunState *st = z.state;
            st->last = z.itmax - 1;
            st->status = kRunGoing;
            st->k = 0;
            st->ticket = 0u;
            st->est[0] = 0.0;
            st->est[1] = INFINITY;
            st->est[2] = NAN;
        }
        *bounds = E;
        __syncthreads();
        return false;
    }

    // ended by the decision of an earlier launch (this one's own sets last to
    // iter - 1, which every workgroup finds out by itself below)
    const int it = (int)a.iter - 1;  // the pass the steps follow
    if (it > 0 && *(volatile const int32_t *)&z.state->last < it) return true;
    clear_next();
    const int axes = z.refine ? (a.one_d ? 1 : D) : 0;
    const int bins = axes * nb;
    for (int e = tid; e < total; e += nthr) prev[e] = a.grid[e];
    for (int e = tid; e < bins; e += nthr) {
        double s = 0.0, c = 0.0;
#pragma unroll
        for (int x = 0; x < kFusedAccs; ++x) two_sum_merge(s, c, z.prev_acc[(size_t)x * a.hist_stride + e], 0.0);
        C[e] = s + c;
    }
    if (wave == waves - 1) {
        // the last wave: the previous pass's totals and the decision after it
        int32_t status = *z.prev_flag != 0u ? kRunNonFinite : kRunGoing;
        if (first_wg || z.tau_rel > 0.0) {
            double sI = 0.0, cI = 0.0, sV = 0.0, cV = 0.0;
            for (int w = lane; w < z.prev_blocks; w += 64) {
                const double *o = z.prev_partials + 4 * (size_t)w;
                two_sum_merge(sI, cI, o[0], o[1]);
                two_sum_merge(sV, cV, o[2], o[3]);
            }
            double Ii = 0.0, Vi = 0.0;  // lane i: pass i
            if (z.tau_rel > 0.0 && lane < it) {
                Ii = z.iters[lane];
                Vi = z.iters[z.itmax + lane];
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const double s2 = __shfl_xor(sI, off, 64), c2 = __shfl_xor(cI, off, 64);
                const double v2 = __shfl_xor(sV, off, 64), e2 = __shfl_xor(cV, off, 64);
                two_sum_merge(sI, cI, s2, c2);
                two_sum_merge(sV, cV, v2, e2);
            }
            const double I = sI + cI, V = sV + cV;
            if (first_wg && lane == 0) {
                z.iters[it] = I;
                z.iters[z.itmax + it] = V;
                // how far the run is, for the host to queue more passes
                if (z.tau_rel > 0.0) *(volatile int32_t *)&z.host->k = it + 1;
            }
            if (z.tau_rel > 0.0 && status == kRunGoing) {
                double est[3];
                wave_weighted_estimate(it + 1, lane < it ? Ii : I, lane < it ? Vi : V, est);
                if (converged_after(it + 1, est, z.tau_rel, z.chi2_max)) status = kRunConverged;
                if (lane == 0)
                    for (int i = 0; i < 3; ++i) est_s[i] = est[i];
            }
        }
        if (lane == 0) status_s = status;
    }
    __syncthreads();
    const int32_t status = status_s;
    if (status != kRunGoing && !first_wg) {
        leave(a, &last_wg);
        return true;
    }
    if (axes) {
        // three-point smoothing (two points at the ends)
        for (int e = tid; e < bins; e += nthr) {
            const int i = e - nb * row_of(e, inv_nb);
            double s;
            if (i == 0) s = (C[e] + C[e + 1]) / 2.0;
            else if (i == nb - 1) s = (C[e - 1] + C[e]) / 2.0;
            else s = ((C[e - 1] + C[e]) + C[e + 1]) / 3.0;
            r[e] = s;
        }
        __syncthreads();
        for (int j = wave; j < axes; j += waves) {
            int b0, b1;
            lane_run(0, nb, lane, &b0, &b1);
            double s = 0.0;
            for (int i = b0; i < b1; ++i) s = s + r[j * nb + i];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) s = s + __shfl_xor(s, off, 64);
            if (lane == 0) axis_sum[j] = s;
        }
        __syncthreads();
        // Lepage's damped compression of each bin's share
        for (int e = tid; e < bins; e += nthr) {
            const double S = axis_sum[row_of(e, inv_nb)];
            if (S > 0.0 && isfinite(S)) r[e] = compressed_share<true>(r[e], S, z.alpha);
        }
        __syncthreads();
        // running sums, made non-decreasing: P[0] = 0, P[i + 1] = r[0] + ... + r[i]
        for (int j = wave; j < axes; j += waves) {
            const double *x = r + j * nb;
            double *Pj = P + j * row;
            int b0, b1;
            lane_run(0, nb, lane, &b0, &b1);
            double s = 0.0;
            for (int i = b0; i < b1; ++i) s = s + x[i];
            double incl = s;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const double y = __shfl_up(incl, off, 64);
                if (lane >= off) incl = incl + y;
            }
            const double left = __shfl_up(incl, 1, 64);
            double run = lane > 0 ? left : 0.0;
            for (int i = b0; i < b1; ++i) {
                run = run + x[i];
                Pj[i + 1] = run;
            }
            if (lane == 0) Pj[0] = 0.0;
            __threadfence_block();
            wave_running_max(Pj, 1, nb + 1, 0.0, lane);
        }
        __syncthreads();
        // boundary k closes k equal shares of the compressed weight (see adjust_axis)
        for (int e = tid; e < bins; e += nthr) {
            const int j = row_of(e, inv_nb), k = e - j * nb;
            const double S = axis_sum[j], *Pj = P + j * row, *Bj = prev + j * row;
            double edge;
            if (!(S > 0.0 && isfinite(S) && Pj[nb] > 0.0)) {
                edge = Bj[k];  // no usable weight: the axis keeps its boundaries
            } else if (k == 0) {
                edge = 0.0;
            } else {
                const double goal = (double)k * (Pj[nb] / (double)nb);
                int lo = 0, hi = nb - 1;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (Pj[mid + 1] < goal) lo = mid + 1;
                    else hi = mid;
                }
                const double rs = r[j * nb + lo];
                double frac = rs > 0.0 ? (goal - Pj[lo]) / rs : 0.0;
                frac = fmin(fmax(frac, 0.0), 1.0);
                edge = __fma_rn(frac, Bj[lo + 1] - Bj[lo], Bj[lo]);
            }
            E[j * row + k] = edge;
            if (k == nb - 1) E[j * row + nb] = 1.0;
        }
        __syncthreads();
        // boundaries never decrease (the first at least the old lower end)
        for (int j = wave; j < axes; j += waves) wave_running_max(E + j * row, 1, nb, prev[j * row], lane);
        __syncthreads();
        if (a.one_d) {  // axis 0's boundaries on every axis
            for (int e = row + tid; e < total; e += nthr) E[e] = E[e - row * row_of(e, inv_row)];
            __syncthreads();
        }
    }
    const double *B = axes ? E : prev;
    if (first_wg) {
        if (axes)
            for (int e = tid; e < total; e += nthr) z.next_grid[e] = B[e];
        if (status != kRunGoing) {
            if (z.host_grid)
                for (int e = tid; e < total; e += nthr) z.host_grid[e] = B[e];
            for (int i = tid; i <= it; i += nthr) {
                z.host_iters[i] = z.iters[i];
                z.host_iters[z.itmax + i] = z.iters[z.itmax + i];
            }
            if (tid == 0) {
                z.state->last = it;
                z.state->status = status;
                for (int i = 0; i < 3; ++i) z.host->est[i] = est_s[i];
                z.host->k = it + 1;
                __threadfence_system();
                *(volatile int32_t *)&z.host->status = status;
            }
            leave(a, &last_wg);
            return true;
        }
    }
    *bounds = B;
    return false;
}

}  // namespace fused
}  // namespace mcubes
