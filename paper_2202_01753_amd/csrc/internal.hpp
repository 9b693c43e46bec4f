// Internal interface between the host driver (mcubes_api.cpp) and the HIP
// kernels (vsample_*.hip, finalize.hip, steps.hip).  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mcubes.h"

namespace mcubes {

constexpr int kMaxDim = 16;
constexpr int kTableN = 256;
constexpr int kMaxBlock = 1024;
constexpr int kBatchBlock = 256;     // threads per workgroup of the batched kernel (or twice that)
constexpr int kBatchMaxBlock = 512;
constexpr int kBatchMaxDim = 10;     // dimensions the batched kernel supports

// A run whose steps between sampling passes (Weighted-Estimates,
// Check-Convergence, Adjust-Bin-Bounds of Alg. 2) run on the device: its
// state in the workspace, mirrored after every pass into page-locked host
// memory that the host reads once the pass is over.  last is the index of
// the run's last iteration: itmax - 1 until a pass ends the run earlier
// (converged, or a non-finite value); every kernel of a later pass then does
// nothing.
struct RunState {
    int32_t last;
    int32_t status;   // kRunGoing, kRunConverged or kRunNonFinite
    int32_t k;        // passes finished
    uint32_t ticket;  // (fused runs) workgroups that are through with the pass that ended the run
    double est[3];    // weighted estimate, its standard deviation, chi^2/dof after k passes
    double pad2;
};
constexpr int32_t kRunGoing = 0, kRunConverged = 1, kRunNonFinite = 2;

// The steps of Alg. 2 before a pass inside its own sampling launch (fused
// runs): every workgroup adjusts the grid from the previous pass's histogram
// by itself, into its LDS, and decides for itself whether the run has ended,
// from the same data in the same order; workgroup 0 also writes both down.
// A pass then costs one launch instead of two and nothing of the grid goes
// through memory between the steps and the pass.  Pass n adds its
// histogram into accumulator set n mod 3, reads set n-1 and clears set n+1 (which
// pass n-1 read), and likewise its totals (two sets) and non-finite flag.  A run
// finds set 0 and flag 0 clear and leaves them so; the others it clears itself.
struct FusedArgs {
    int32_t refine;         // the previous pass collected contributions: adjust the grid
    int32_t prev_blocks;    // workgroups of the previous pass (0: this is the first pass)
    int32_t itmax;
    const double *prev_partials;
    double *prev_acc, *clear_acc;
    uint32_t *prev_flag, *clear_flag;
    double *next_grid;      // the adjusted grid (first pass: equal bins), written by workgroup 0
    RunState *state;        // run state; iters after it
    double *iters;
    RunState *host;         // host mirror, its iters and grid (grid may be null)
    double *host_iters, *host_grid;
    double tau_rel, chi2_max, alpha;
};
// Up to which size a run is fused: bins (every workgroup adjusts all axes),
// passes (one lane of a wave each) and samples per pass.  Per pass, steps in a
// launch of their own against fused: d = 2, 1e4 samples, 100 bins 21.7 -> 14.9 us;
// d = 3, 1e6, 500 bins 32.4 -> 30.3; d = 8, 1e5, 100 bins, FP32 25.4 -> 22.7;
// d = 10, 1e6, 100 bins 39.7 -> 37.7; but d = 10, 5e5, 200 bins 34.3 -> 34.6, d = 6,
// 4e6, 100 bins 51.5 -> 51.5 and d = 4, 8e6, 100 bins, FP32 54.3 -> 57.4.
constexpr int kFusedMaxBins = 1600;
// The same for runs to a target, which may end after two passes and then have paid
// every axis's steps in every workgroup three times.  Whole runs at 1e4, 1e5 and 1e6
// samples (FP64), fused against launches of their own, of two passes: 100 bins 59, 68
// and 85 us against 72, 69 and 75; 200 bins 65, 74, 87 against 69, 69, 75; 300 (d = 5)
// 71, 76, 92 against 67, 68, 79; 600 (d = 5) 78, 82, 95 against 69, 69, 80.  Of twelve passes:
// 100 bins 195, 234, 285 against 262, 259, 295; 200 bins 209, 238, 292 against 252, 259,
// 303; 300 (d = 5) 236, 249, 327 against 264, 266, 323; 600 (d = 5) 267, 275, 338 against
// 269, 273, 335.
constexpr int kFusedTargetBins = 200;
constexpr int kFusedMaxPasses = 64;
constexpr int64_t kFusedMaxSamples = int64_t(1) << 22;
// Accumulators in use of each set: every workgroup reads them all before it
// can sample (two instead of kHistAcc: d = 8, 1e5 samples 27.9 instead of 32.9 us
// per pass; one: 28.9, for the additions that then meet in it).
constexpr int kFusedAccs = 2;
// Doubles of LDS the steps inside a launch need after the grid: C/E, r, P and
// the old boundaries (d rows of nb + 1 each).
constexpr size_t fused_scratch(int d, int nb) { return 4 * (size_t)d * (nb + 1); }

// Everything the sampling kernel needs, passed by value so that the per-axis
// constants arrive in scalar registers.
struct SampleArgs {
    const double *grid;     // dim*(nb+1) boundaries, unit coordinates
    const void *tables;     // the two tables in the device layout of the evaluation precision
                            // (see table_cell), or nullptr
    double *partials;       // per workgroup 4 totals
    double *hist_acc;       // kHistAcc histogram accumulators, hist_stride doubles apart
    uint32_t *flag;         // set to nonzero when the integrand is not finite
    double *trace;          // optional per-sample / per-cube records
    int64_t m;              // sub-cubes
    int64_t t0, t1;         // traced sub-cube range
    int64_t stride;         // sub-cubes advanced per lane step (= grid size in threads)
    uint64_t seed;
    uint64_t gmagic;        // ceil(2^64 / g) (0 for g = 1): quotients of 32-bit indices by g
    uint32_t iter;
    int32_t p;              // samples per sub-cube
    int32_t nb;             // bins per axis
    int32_t g;              // intervals per axis
    int32_t hist;           // nonzero: collect bin contributions (V-Sample)
    int32_t hist_stride;    // doubles between two histogram accumulators
    int32_t kind;           // integrand id * 32 + dim (dispatch in the batched kernel)
    int32_t one_d;          // nonzero: collect bin contributions of the first axis only
    int32_t hist_copies;    // LDS histogram copies.  kPlain: 2 = lanes 32-63 of a wave add into a
                            // second; kCopies, kSplit: 2^copy_shift, side by side per bin
    int32_t copy_shift;
    int32_t window;         // kStaged: bins a stratum of a slow axis can reach, at most
    int32_t stage_shift;    // kStaged: log2 of the copies of a window's bins (2 to 5)
    uint32_t block_cubes;   // kStaged: sub-cubes per block of the fast axes, g^K
    uint32_t blocks_total;  // and blocks, g^NS
    int32_t lsplit;         // kSplit: a sub-cube's samples go over 2^lsplit neighbouring lanes
    double s;               // nb / g
    float s32;              // nb / g rounded to float (FP32 evaluation)
    int32_t fp32;           // nonzero: FP32 evaluation
    double j0;              // FP64: the volume times nb^dim, the Jacobian's first factor
    double inv;             // 1 / (m p)
    double pd;              // p
    double inv_pm1;         // 1 / (p - 1)
    double cval;            // constant integrand value
    const void *consts;     // kConstStride values of the evaluation precision per axis
    const int32_t *run_last;  // nullptr, or the last iteration of a run whose steps run on the
                              // device: a pass with iter beyond it does nothing
    int32_t sdig[kMaxDim];  // stride in base g, least significant digit first
    FusedArgs fused;        // kFused
};

// Per-axis constants, in device memory (the kernels read them with scalar loads):
//   [0] lo   [1] span = hi - lo   [2] q = nb * span
//   [3] Gaussian centre or corner-peak coefficient   [4] Gaussian 1/width   [5] 0
constexpr int kConstStride = 6;

// The sampling kernels of one integrand, dimension and precision.
constexpr int kPlain = 0;   // one lane per sub-cube
constexpr int kTraced = 1;  // kPlain with per-sample and per-cube records
constexpr int kCopies = 2;  // 2^copy_shift copies of every histogram bin side by side
constexpr int kSplit = 3;   // kCopies, and a sub-cube's samples over 2^lsplit neighbouring lanes
constexpr int kFused = 4;   // kSplit (lsplit may be 0) with the steps before the pass inside (FusedArgs)
constexpr int kStaged = 5;  // blocks of sub-cubes that share their slow axes' digits (adjusting passes)
constexpr int kStagedUnit = 6;  // kStaged on the unit cube, whose points need no scaling
constexpr int kPerAxis = 7;  // kPlain whose Jacobian is multiplied axis by axis (FP64): see first_jacobian
// The slow axes of the staged kernels of a dimension (0: there is none).
constexpr int staged_slow_axes(int integrand, int dim) {
    return integrand == 0 ? 0 : dim == 5 || dim == 6 ? 2 : dim == 7 ? 3 : dim >= 8 && dim <= 10 ? 4 : 0;
}
// Waves per SIMD they are compiled for and launched at: six (two workgroups of
// 768 threads per CU) in FP32 evaluation, one sample at a time, for the FP64
// corner peak and the FP64 Gaussian at d = 5, which fit 80 registers without
// spills; four (one of 1024) for the others.
constexpr int staged_waves(int integrand, int dim, bool fp32) {
    return fp32 || integrand == MC_F_CORNER_PEAK || (integrand == MC_F_GAUSS_PRODUCT && dim == 5) ? 6 : 4;
}

// Which of them a pass of the problem takes (adjust 1 or 0), or with run set the
// passes of a whole run with the steps on the device: kFused, or the passes'
// own; -1 for an invalid problem.  For the tests; not part of the C ABI.
extern "C" int32_t mcubes_launch_kind(const mc_problem *prob, int32_t adjust, int32_t run);

// The sampling kernel of that kind, or nullptr.
const void *sample_kernel(int integrand, int dim, int kind, bool fp32);

// Launches a sampling kernel; lds_bytes is the dynamic LDS size.
hipError_t launch_sample(const void *kernel, int blocks, int threads, size_t lds_bytes, hipStream_t stream,
                         const SampleArgs &args);

// Histogram accumulators of a V-Sample pass (a region of their own, so that
// the totals of a pass with more workgroups never reach them): workgroup b
// adds its LDS histogram into accumulator b % kHistAcc with device-scope
// FP64 atomics.  Eight copies cut the atomics that meet on one address
// eightfold (workgroups are dispatched round-robin over the chip's eight
// XCDs, so the copies also split by XCD); they are summed in order after the
// pass, by the finalize or by the steps kernel.
constexpr int kHistAcc = 8;

// Reduces the per-workgroup totals in a fixed order and sums the histogram
// accumulators in order into out = [I, var, flag, 0, hist...]; clears the
// accumulators (for the next pass) and the flag.  (Runs whose steps between
// passes are on the host.)  With a counter in device memory (zero), out and
// done are mapped host memory, and seq is written to *done once out is whole.
hipError_t launch_finalize(const double *partials, double *hist_acc, int blocks, int nhist, int hist_stride,
                           int with_hist, uint32_t *flag, double *out, uint32_t *counter, uint32_t *done,
                           uint32_t seq, hipStream_t stream);

// n doubles from mapped host memory src into device memory dst.
hipError_t launch_upload(const double *src, double *dst, int n, hipStream_t stream);

// The decision after pass it of such a run.  iters holds I_0 .. I_{itmax-1},
// then var_0 .. var_{itmax-1}, on the device; host_iters the same in the host
// mirror (host, host_iters: mapped page-locked memory).
struct RunCtl {
    RunState *state;
    double *iters;
    RunState *host;
    double *host_iters;
    int32_t it, itmax;
    double tau_rel, chi2_max;
    int32_t all;              // nonzero: mirror every pass's results, not this one's alone
};

// Start of a device-steps run: the state (last = itmax - 1, nothing done) and
// Init-Bins (boundaries i/nb on every axis) in the workspace, and in
// host_grid (mapped host memory) unless it is null.
hipError_t launch_run_init(RunState *state, double *grid, double *host_grid, int d, int nb, int itmax,
                           hipStream_t stream);

// Everything between pass ctl.it and the next of a device-steps run, one
// launch: the totals merged and the decision taken (ctl), and in an
// adjusting pass (nref = d, or 1 for m-Cubes1D; 0 otherwise) the grid
// adjusted from the histogram accumulators, one workgroup per axis.
struct StepsArgs {
    RunCtl ctl;
    const double *partials;   // the pass's per-workgroup totals
    int32_t blocks;           // workgroups of the pass
    int32_t hist_stride;
    double *hist_acc;         // kHistAcc accumulators, or kFusedAccs at the end of a fused run (cleared
                              // as they are read)
    uint32_t *flag;           // non-finite flag (read and cleared)
    double *grid;             // d*(nb+1) boundaries, adjusted in place
    double *host_grid;        // mapped host copy of the boundaries, or null
    double alpha;
    int32_t d, nb, one_d, nref;
    // end of a fused run: the accumulator set and flag that its last pass read,
    // to be cleared, and the grid mirrored whether it was adjusted or not
    double *clear_acc;        // or null
    uint32_t *clear_flag;
};
hipError_t launch_steps(const StepsArgs &args, hipStream_t stream);

// Adjust-Bin-Bounds on the device (mc_refine_grid_device): one workgroup per
// axis (m-Cubes1D: axis 0, then copied to every axis), the host's steps with
// sums in a fixed order of its own and the device library's pow and log: the
// host's result to rounding.  Reads the histogram hist (d*nb), rewrites grid
// in place.
hipError_t launch_refine(double *grid, const double *hist, int d, int nb, int one_d, double alpha,
                         hipStream_t stream);
// LDS of one adjusting workgroup, and the largest nb it takes.
size_t refine_lds_bytes(int nb);
constexpr int kDeviceStepsMaxBins = MC_DEVICE_STEPS_MAX_BINS;

// Zeroes n doubles (the histogram accumulators, before a workspace's first pass).
hipError_t launch_zero(double *p, size_t n, hipStream_t stream);

// ---- batched sampling: many integrals in one persistent launch ----

// One integral of a batch.  a carries its constants, grid and table pointers,
// lattice, iteration and whether this pass collects bin contributions (its
// trace, partials and stride fields are unused).  out holds [I, var, flag, 0,
// d*nb bin contributions] of the integral's latest pass: the segments add
// their bin contributions into it (zero at admission and after every bin
// adjustment); when refine is set, the grid is adjusted on the device from
// that histogram after the pass.
//
// Each integral also keeps on the device the results of all its iterations
// (iters: I_0.. I_{itmax-1}, then var_0 .. var_{itmax-1}) and a state word:
// the merge kernel runs Weighted-Estimates and Check-Convergence after every
// pass and sets the state once the integral stops (converged, out of
// iterations, or a non-finite value).  Later steps may still list it (the
// host learns of the stop one step later); its segments then do no work.
struct BatchItem {
    SampleArgs a;
    double *grid;       // the integral's grid (a.grid, writable)
    double *out;
    double *iters;      // 2 * itmax doubles
    uint32_t *state;    // kItemRunning until the integral stops
    double alpha;
    double tau_rel;     // Check-Convergence: target relative error (0: never converged)
    double chi2_max;    //   and bound on chi^2/dof (0: default, negative: unchecked)
    int32_t itmax;
    int32_t refine;
};

// Item states, and the merge kernel's per-step results (kResStride doubles
// per listed integral: I, var, non-finite flag, weighted estimate, its
// standard deviation, chi^2/dof, state after the pass or kResSkipped, 1 if
// converged).
constexpr uint32_t kItemRunning = 0, kItemDone = 1, kItemFailed = 2;
constexpr int kResStride = 8;
constexpr double kResSkipped = -1.0;

// A contiguous range of one integral's sub-cubes, processed by one workgroup.
struct BatchSegment {
    int32_t item;       // integral (index into the items array)
    int32_t pad;
    int64_t t0, t1;     // sub-cubes [t0, t1)
};

// The device arrays of one batched step.  An integral's segments are
// contiguous, [item_first[i], item_first[i+1]).  The workgroups of one
// launch take the segments order[lo], order[lo+1], ... one at a time from the
// launch's counter *queue (zero before the step) until it reaches hi.
struct BatchArgs {
    const BatchItem *items;
    const BatchSegment *segs;
    const int32_t *order;
    const int32_t *item_first;
    double *seg_tot;          // 4 doubles per segment
    uint32_t *flags;          // per item, zero before the step
    double *res;              // per item: kResStride doubles (packed for one read-back)
    uint32_t *queue;          // this launch's segment counter
    int32_t lo, hi;           // this launch's range of order
    int32_t n_items;
};

// Admission of one integral into a batch: its per-axis constants are copied
// from the step's upload into its block, its starting grid (Init-Bins,
// uniform boundaries i/nb on every axis) is written there and its output
// (totals and bin contributions) is cleared.
struct AdmitRecord {
    char *consts;         // destination of the constants in the integral's block
    double *grid;         // destination of the d*(nb+1) starting boundaries
    double *out;          // the integral's 4 + d*nb output doubles
    uint32_t *state;      // the integral's state word (set to kItemRunning)
    int64_t src;          // byte offset of the constants in the upload (4-byte aligned)
    int32_t const_words;  // 4-byte words of constants
    int32_t dim, nb, pad;
};
hipError_t launch_admit(const AdmitRecord *recs, int n, const char *upload, hipStream_t stream);

// Launches the batched sampling kernel of one precision and integrand family
// (tables: the Gaussian-times-tables integrand; otherwise the closed-form
// ones) over the segments order[args.lo .. args.hi) (args.queue is this
// launch's counter).  threads is kBatchBlock or kBatchMaxBlock.
hipError_t launch_batch(bool fp32, bool tables, int blocks, int threads, size_t lds_bytes,
                        hipStream_t stream, const BatchArgs &args);
const void *batch_kernel(bool fp32, bool tables);
// Merges every running integral's segment totals in order into its out and
// res, clears its flag, appends (I, var) to its iterations and decides
// whether it stops (Weighted-Estimates, Check-Convergence, itmax).
hipError_t launch_batch_finalize(const BatchArgs &args, hipStream_t stream);
// Adjust-Bin-Bounds on the device for n_axes (integral, axis) pairs
// (axis_item[2a], axis_item[2a+1]): reads the integral's histogram row from its
// out (and clears it for the next collecting pass) and its boundaries from
// a.grid, writes the new ones to next_grid[integral].
hipError_t launch_batch_refine(const BatchItem *items, const int32_t *axis_item,
                               double *const *next_grid, int n_axes, int max_nb,
                               hipStream_t stream);

}  // namespace mcubes
