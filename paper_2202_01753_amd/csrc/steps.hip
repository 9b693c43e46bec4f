// The steps of Alg. 2 between two sampling passes, on the device, for runs
// that keep them there: the start of a run (Init-Bins and the run state), and
// after each pass one launch that merges the pass's results, runs
// Weighted-Estimates and Check-Convergence, and Adjust-Bin-Bounds.
//
// The bin adjustment takes the host's steps (three-point smoothing, Lepage's
// damped compression, equal shares of the compressed weight per new bin)
// with the same comparisons and the same interpolation, one workgroup per
// axis.  Its sums are formed in a fixed order of its own (each thread a
// contiguous run of bins, then across the threads) rather than the host's
// one bin after another, and pow and log are the device library's, so the
// boundaries agree with the host's to rounding, not bit for bit; the result
// does not depend on timing.  Each new boundary is found by its own thread,
// with a binary search over the running sums for the bin where the host's
// scan would stop.
#include <cmath>

#include "adjust.hpp"
#include "estimate_device.hpp"
#include "internal.hpp"
#include "merge.hpp"

namespace mcubes {

namespace {

static_assert(kRefineThreads == merge::kThreads, "the steps kernel's last workgroup merges the totals");

__global__ void __launch_bounds__(256) run_init_kernel(RunState *st, double *grid, double *host_grid, int d,
                                                       int nb, int itmax) {
    const int row = nb + 1;
    for (int i = threadIdx.x; i < d * row; i += blockDim.x) {
        const double b = (double)(i % row) / (double)nb;
        grid[i] = b;
        if (host_grid) host_grid[i] = b;
    }
    if (threadIdx.x == 0) {
        st->last = itmax - 1;
        st->status = kRunGoing;
        st->k = 0;
        st->ticket = 0u;
        st->est[0] = 0.0;
        st->est[1] = INFINITY;
        st->est[2] = NAN;
        st->pad2 = 0.0;
    }
    if (host_grid) __threadfence_system();
}

// Adjust-Bin-Bounds of axis j: grid row j is rewritten in place (m-Cubes1D, j = 0:
// and copied to every axis); host_grid, if not null, receives every boundary
// written to grid, and with mirror_unmoved also those of an axis that keeps
// its boundaries (the host copy holds nothing yet).
__device__ __forceinline__ void adjust_axis(double *lds, const double *C, double *grid, double *host_grid, int j,
                                            int d, int nb, int one_d, double alpha, bool mirror_unmoved) {
    const int tid = threadIdx.x;
    double *B = grid + (size_t)j * (nb + 1), *H = host_grid ? host_grid + (size_t)j * (nb + 1) : nullptr;
    const double *prev = lds + 2 * (size_t)nb + 1, *src = adjusted_axis<false>(lds, C, B, nb, alpha);
    const bool moved = src != prev;
    for (int i = tid; i <= nb; i += kRefineThreads) {
        if (moved) B[i] = src[i];
        if (H && (moved || mirror_unmoved)) H[i] = src[i];
    }
    // m-Cubes1D: axis 0's boundaries, adjusted or not, on every axis
    if (one_d)
        for (int c = 1; c < d; ++c)
            for (int i = tid; i <= nb; i += kRefineThreads) {
                B[(size_t)c * (nb + 1) + i] = src[i];
                if (H) H[(size_t)c * (nb + 1) + i] = src[i];
            }
    if (host_grid) __threadfence_system();
}

// mc_refine_grid_device: one workgroup per axis (m-Cubes1D: one), the
// contributions read from hist.
__global__ void __launch_bounds__(kRefineThreads)
refine_kernel(double *grid, const double *hist, int d, int nb, int one_d, double alpha) {
    extern __shared__ double lds[];
    adjust_axis(lds, hist + (size_t)blockIdx.x * nb, grid, nullptr, blockIdx.x, d, nb, one_d, alpha, false);
}

// Everything between pass it and the next of a device-steps run, in one
// launch (nothing once the run has ended before pass it).  Workgroups
// [0, nref) adjust one axis each (nref = 0 in a No-Adjust pass), taking the
// axis's contributions from the histogram accumulators (summed in order and
// cleared, as the finalize does); workgroup nref merges the totals and takes
// the pass's decision.  The adjustment of pass it does not depend on that
// decision (a run refines after its last adjusting pass too).
__global__ void __launch_bounds__(kRefineThreads) steps_kernel(const StepsArgs A) {
    if (A.ctl.it > A.ctl.state->last) return;  // (this launch sets last to it at most)
    extern __shared__ double lds[];
    if ((int)blockIdx.x < A.nref) {
        const int j = blockIdx.x, nb = A.nb;
        double *C = lds + 3 * (size_t)nb + 2;  // the E array, free until the search
        for (int i = threadIdx.x; i < nb; i += kRefineThreads)
            C[i] = A.clear_acc ? merge::take_bin<kFusedAccs>(A.hist_acc, (size_t)j * nb + i, A.hist_stride)
                               : merge::take_bin<kHistAcc>(A.hist_acc, (size_t)j * nb + i, A.hist_stride);
        __syncthreads();
        adjust_axis(lds, C, A.grid, A.host_grid, j, A.d, nb, A.one_d, A.alpha, A.clear_acc != nullptr);
        return;
    }
    if (A.clear_acc) {
        for (int i = threadIdx.x; i < kFusedAccs * A.hist_stride; i += kRefineThreads) A.clear_acc[i] = 0.0;
        if (threadIdx.x == 0) *A.clear_flag = 0u;
        if (A.nref == 0 && A.host_grid)
            for (int i = threadIdx.x; i < A.d * (A.nb + 1); i += kRefineThreads) A.host_grid[i] = A.grid[i];
    }
    double I = 0.0, V = 0.0;
    merge::pass_totals(A.partials, A.blocks, &I, &V);
    if (threadIdx.x < 64) {
        const bool bad = *A.flag != 0u;
        if (threadIdx.x == 0) *A.flag = 0u;
        merge::decide(A.ctl, I, V, bad);
    }
}

}  // namespace

size_t refine_lds_bytes(int nb) { return sizeof(double) * (4 * (size_t)nb + 3); }

hipError_t launch_run_init(RunState *state, double *grid, double *host_grid, int d, int nb, int itmax,
                           hipStream_t stream) {
    hipLaunchKernelGGL(run_init_kernel, dim3(1), dim3(256), 0, stream, state, grid, host_grid, d, nb,
                       itmax);
    return hipGetLastError();
}

hipError_t launch_refine(double *grid, const double *hist, int d, int nb, int one_d, double alpha,
                         hipStream_t stream) {
    const size_t lds = refine_lds_bytes(nb);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&refine_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(refine_kernel, dim3(one_d ? 1 : d), dim3(kRefineThreads), lds, stream, grid,
                       hist, d, nb, one_d, alpha);
    return hipGetLastError();
}

hipError_t launch_steps(const StepsArgs &args, hipStream_t stream) {
    const size_t lds = args.nref ? refine_lds_bytes(args.nb) : 0;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&steps_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(steps_kernel, dim3(args.nref + 1), dim3(kRefineThreads), lds, stream, args);
    return hipGetLastError();
}

}  // namespace mcubes
