// Host side of the m-Cubes library: validation, the sub-cube lattice, the
// workspace layout, the per-iteration host steps of Alg. 2 (weighted
// estimate, bin adjustment, convergence check) and the C ABI.
//
// Built without floating-point contraction: the bin adjustment must round
// exactly as written so that a given histogram always yields the same grid.
#include "mcubes.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

#include "host.hpp"
#include "host_pool.hpp"
#include "internal.hpp"

using namespace mcubes;
using namespace mcubes::host;

namespace {


// ------------------------------------------------------------------ launch geometry and workspace

constexpr size_t kFlagBytes = 64;      // three flags and the finalize's counter, a whole number of doubles
constexpr size_t kCounterOffset = 32;

// A sampling launch: which kernel, its shape in adjusting and No-Adjust passes.
struct Launch {
    int kind;                 // kPlain, kTraced, ...
    const void *fn;
    int threads;
    int blocks_adj, blocks_noadj;
    size_t lds_adj, lds_noadj;
    int hist_copies;          // LDS histogram copies in adjusting passes
    int copy_shift, lsplit;   // kCopies, kSplit: log2 of the copies, of the lanes per sub-cube
    int window, stage_shift;  // kStaged: bins of a slow axis's window, log2 of their copies
    int blocks(bool adjust) const { return adjust ? blocks_adj : blocks_noadj; }
    size_t lds(bool adjust) const { return adjust ? lds_adj : lds_noadj; }
};

struct Geometry {
    int64_t g, m, p;
    Launch adj, noadj, traced;  // of adjusting and No-Adjust passes, and of traced ones of either
    const Launch &pass(bool adjust) const { return adjust ? adj : noadj; }
    int hist_stride;          // doubles per histogram accumulator (padded)
    bool fusable;             // runs may have their steps inside the sampling launches
    size_t off_consts, off_grid, off_tables, off_hist, off_flag, off_out, off_run, off_partials, off_fused_grid,
        off_fused_hist, off_fused_partials;
    size_t total;
    // accumulator set, non-finite flag, totals and grid of pass n in a fused
    // run (the first of each in others)
    size_t hist_set(int n) const {
        return n % 3 ? off_fused_hist + sizeof(double) * kFusedAccs * (size_t)hist_stride * (n % 3 - 1) : off_hist;
    }
    size_t flag_set(int n) const { return off_flag + sizeof(uint32_t) * (n % 3); }
    size_t partials_set(int n) const { return n % 2 ? off_fused_partials : off_partials; }
    size_t grid_set(int n) const { return n % 2 ? off_fused_grid : off_grid; }
};

mc_status blocks_for(const void *fn, int threads, size_t lds, int64_t m, int requested, int *out) {
    int cus = 0, per_cu = 0;
    HIP_TRY(compute_units(&cus));
    HIP_TRY(allow_lds(fn, lds));
    HIP_TRY(occupancy(fn, threads, lds, &per_cu));
    if (per_cu < 1) return MC_EINVAL;
    // Where several workgroups share a CU, launch more than fit at once: the
    // workgroups are smaller, and CUs that were handed fewer of them take more
    // later, instead of idling for the rest of the launch (four times as many:
    // 12% faster at d = 8 with two 768-thread workgroups per CU; one 1024-thread
    // workgroup per CU gains nothing and keeps the resident count).  Every
    // workgroup also ends with a flush of its histogram, so four times is
    // taken only where each lane still has at least 100 sub-cubes to do,
    // twice otherwise (the FP32 d = 6 tables pass: 60 per lane at twice;
    // once, twice and four times measured 0.632, 0.615 and 0.616 ms).
    const int64_t resident = (int64_t)per_cu * cus;
    int64_t want = resident;
    if (requested > 0)
        want = requested;
    else if (per_cu > 1)
        want = m >= (int64_t)100 * 4 * resident * threads ? 4 * resident : 2 * resident;
    const int64_t useful = (m + threads - 1) / threads;
    if (requested <= 0) want = std::min(want, useful);
    *out = (int)std::max<int64_t>(1, std::min<int64_t>(want, 1 << 20));
    return MC_OK;
}

// Workgroup size when the problem leaves it open: of 1024, 768, 512 and 256
// threads (whole multiples of four waves, so each of a CU's four SIMDs holds
// the same number of every workgroup's waves), the one that keeps the most
// waves resident given the kernel's registers, the adjusting pass's LDS and the
// workgroups asked for, if any (d = 16 Gaussian, 2e7 samples, FP32, 64
// workgroups, No-Adjust: 1.86 ms with 1024 threads, 2.72 with the 256 that keep most
// resident on a full chip); on a tie the larger, which means fewer workgroups
// and so fewer histogram flushes.  768 is the d = 8 case: two 64 KB
// workgroups of 12 waves fit where one of 16 did.
mc_status pick_threads(const void *fn, size_t lds, int requested, int *out) {
    int cus = 0, best = 0;
    HIP_TRY(compute_units(&cus));
    HIP_TRY(allow_lds(fn, lds));
    int64_t best_waves = -1;
    for (int t : {1024, 768, 512, 256}) {
        int per_cu = 0;
        HIP_TRY(occupancy(fn, t, lds, &per_cu));
        int64_t resident = (int64_t)per_cu * cus;
        if (requested > 0) resident = std::min<int64_t>(resident, requested);
        const int64_t waves = resident * (t / 64);
        if (waves > best_waves) {
            best_waves = waves;
            best = t;
        }
    }
    if (best_waves < 1) return MC_EINVAL;
    *out = best;
    return MC_OK;
}

// The launch of one lane per sub-cube (kPlain or kPerAxis; kTraced in its shape).
mc_status plain_launch(const mc_problem *pr, int kind, int64_t m, Launch *out) {
    const int d = pr->dim, nb = pr->nbins;
    const bool f32 = is_fp32(pr);
    Launch L{};
    L.kind = kind;
    L.fn = sample_kernel(pr->integrand, d, kind, f32);
    if (!L.fn) return MC_EINVAL;
    L.lds_adj = lds_bytes_of(d, nb, true, f32);
    L.lds_noadj = lds_bytes_of(d, nb, false, f32);
    mc_status st;
    if (pr->threads) {
        L.threads = pr->threads;
    } else {
        st = pick_threads(L.fn, L.lds_adj, pr->blocks, &L.threads);
        if (st != MC_OK) return st;
    }
    // A second LDS copy of the histogram, for the upper half of each wave,
    // halves the lanes that add into one bin at once (lanes of a wave share
    // the strata of all but the fastest axes, so many fall into the same few
    // bins); taken where the extra LDS keeps as many workgroups resident.
    L.hist_copies = 1;
    const size_t lds2 = L.lds_adj + sizeof(double) * d * (size_t)nb;
    if (lds2 <= kLdsDynamicLimit) {
        int per1 = 0, per2 = 0;
        HIP_TRY(allow_lds(L.fn, lds2));
        HIP_TRY(occupancy(L.fn, L.threads, L.lds_adj, &per1));
        HIP_TRY(occupancy(L.fn, L.threads, lds2, &per2));
        if (per2 >= per1 && per2 > 0) {
            L.hist_copies = 2;
            L.lds_adj = lds2;
        }
    }
    st = blocks_for(L.fn, L.threads, L.lds_adj, m, pr->blocks, &L.blocks_adj);
    if (st != MC_OK) return st;
    st = blocks_for(L.fn, L.threads, L.lds_noadj, m, pr->blocks, &L.blocks_noadj);
    if (st != MC_OK) return st;
    *out = L;
    return MC_OK;
}

// What a launch with this many waves per CU and histogram copies (1: kPlain,
// with its second copy for half the lanes or not) is worth against others of
// the same problem.  Below 24 waves the kernels cover less of their latency;
// copies side by side take lanes that meet in one bin, or on one LDS bank,
// apart (an FP64 LDS atomic takes 8.7 cycles per wave with 64 different
// banks, 26 at random bins of 500, 33 at random bins of 42, 192 in one bin).
// Measured against kPlain: 4 copies at equal waves 1.04-2.5 times as fast
// (d = 2 to 10, 100 to 500 bins, 1e6 to 1e8 samples), 8 or 16 copies at 16
// waves against 24 1.05-1.39; 4 copies at 16 against 24 0.92-0.96 in FP64 and with
// the tables, whose VALU work leaves the LDS idle at times, and 1.09-1.11 in
// FP32 evaluation of the closed forms, where the LDS sets the pace.
double launch_worth(int waves, int copies, bool lds_bound) {
    const double w = waves >= 24 ? 1.0 : waves >= 20 ? 0.96 : waves >= 16 ? 0.90 : waves / 16.0 * 0.90;
    const double c = copies >= 16 ? 1.05 : copies >= 8 ? 1.03 : copies >= 4 ? (lds_bound ? 1.0 : 0.95) : 0.87;
    return w * c;
}

// The launch with several copies of the histogram side by side (kCopies) and,
// where there are fewer sub-cubes than lanes, a sub-cube's samples over
// several lanes (kSplit), where it is worth more than the plain one, which
// *out holds on entry.
mc_status copies_launch(const mc_problem *pr, int64_t g, int64_t m, int64_t p, const Launch &plain, Launch *out) {
    const int d = pr->dim, nb = pr->nbins;
    const bool f32 = is_fp32(pr);
    const size_t grid = lds_bytes_of(d, nb, false, f32), one = sizeof(double) * d * (size_t)nb;
    const bool lds_bound = f32 && pr->integrand != MC_F_GAUSS_TABLES;
    int cus = 0, per_cu = 0;
    HIP_TRY(compute_units(&cus));
    HIP_TRY(occupancy(plain.fn, plain.threads, plain.lds_adj, &per_cu));
    const double plain_worth = launch_worth(per_cu * plain.threads / 64, 1, lds_bound);
    Launch L{};
    L.kind = kCopies;
    L.fn = sample_kernel(pr->integrand, d, kCopies, f32);
    if (!L.fn) return MC_EINVAL;
    double best = 0.0;
    for (int t : {1024, 768, 512, 256}) {
        // (a given number of workgroups keeps the plain launch's threads: smaller
        // ones would leave the problem fewer lanes)
        const bool given = pr->threads || pr->blocks;
        if (given && t != 1024) break;
        const int threads = given ? plain.threads : t;
        for (int cs = 4; cs >= 2; --cs) {
            const size_t lds = grid + (one << cs);
            if (lds > kLdsDynamicLimit) continue;
            HIP_TRY(allow_lds(L.fn, lds));
            HIP_TRY(occupancy(L.fn, threads, lds, &per_cu));
            const double worth = launch_worth(per_cu * threads / 64, 1 << cs, lds_bound);
            if (per_cu > 0 && worth > best) {
                best = worth;
                L.threads = threads;
                L.copy_shift = cs;
            }
        }
    }
    if (best <= plain_worth) return MC_OK;
    // One row of contributions (m-Cubes1D): copies only keep apart the lanes of a
    // wave whose 64 strata of axis 0 lie in fewer than 12 bins (d = 2, 1e8 samples,
    // 100 bins, FP32: 288 us against 517; 1e7, 300 bins, 8.6 bins per wave: 57 against
    // 74); elsewhere their address arithmetic on every axis costs more (d = 8 corner peak,
    // 1e9, FP32: 4950 against 4360 us; d = 4, 4.3e8 1480 against 1344; d = 3, 1e8, 17
    // bins per wave: 318 against 302).  Passes that may be fused keep them.
    if (pr->one_d && m * p > kFusedMaxSamples && 64 * (int64_t)nb >= 12 * g) return MC_OK;
    // Lanes: the resident ones.  Fewer sub-cubes than that: as many lanes per
    // sub-cube as still fit, each with a sample or more to do, and smaller
    // workgroups where the lanes would otherwise fill only some of the CUs
    // (ten axes, 1e6 samples, 59049 sub-cubes of 16 samples: 84 -> 40 us per pass;
    // eight axes, 1e5 samples, 6561 of 15: 47 -> 25 us).
    HIP_TRY(occupancy(L.fn, L.threads, grid + (one << L.copy_shift), &per_cu));
    int64_t resident = (int64_t)per_cu * cus;
    if (pr->blocks) resident = pr->blocks;
    while (L.lsplit < 6 && (2 << L.lsplit) <= p && m <= (resident * L.threads) >> (L.lsplit + 1)) ++L.lsplit;
    const int64_t lanes = m << L.lsplit;
    if (!pr->threads && !pr->blocks) {
        if (lanes <= (int64_t)cus * 256) L.threads = 256;
        else if (lanes <= (int64_t)cus * 512) L.threads = std::min(L.threads, 512);
    }
    if (L.lsplit) {
        L.kind = kSplit;
        L.fn = sample_kernel(pr->integrand, d, kSplit, f32);
        if (!L.fn) return MC_EINVAL;
    }
    const int64_t useful = (lanes + L.threads - 1) / L.threads;
    // clearing and adding up the copies is work per workgroup: no more of them
    // than twice the samples a bin of the workgroup gets
    const int64_t per_wg = m * p / std::max<int64_t>(1, std::min(useful, resident));
    while (L.copy_shift > 0 && ((int64_t)nb << L.copy_shift) > 2 * per_wg) --L.copy_shift;
    L.hist_copies = 1 << L.copy_shift;
    L.lds_noadj = grid;
    L.lds_adj = grid + (one << L.copy_shift);
    for (int adj = 0; adj < 2; ++adj) {
        const size_t lds = adj ? L.lds_adj : L.lds_noadj;
        HIP_TRY(allow_lds(L.fn, lds));
        HIP_TRY(occupancy(L.fn, L.threads, lds, &per_cu));
        if (per_cu < 1) return MC_OK;
        int64_t blocks = pr->blocks ? pr->blocks : std::min((int64_t)per_cu * cus, useful);
        blocks = std::max<int64_t>(1, std::min<int64_t>(blocks, 1 << 20));
        (adj ? L.blocks_adj : L.blocks_noadj) = (int)blocks;
    }
    *out = L;
    return MC_OK;
}

int64_t int_pow(int64_t b, int e) {
    int64_t v = 1;
    for (int i = 0; i < e; ++i) v *= b;
    return v;
}

// The staged launch of an adjusting pass (see vsample_staged_kernel), in place
// of the one *out holds: where the blocks' rounds fill the workgroups (idle
// lanes of a block's last round and unequal shares cost at most what it gains:
// 7% in FP64, 12% in FP32 evaluation) and its LDS leaves as many waves resident.
mc_status staged_launch(const mc_problem *pr, int64_t g, int64_t m, Launch *out) {
    const int d = pr->dim, nb = pr->nbins, ns = staged_slow_axes(pr->integrand, d), K = d - ns;
    const bool f32 = is_fp32(pr);
    if (!ns || g < 2 || m > 0xFFFFFFFFll || pr->one_d || pr->threads || pr->blocks) return MC_OK;
    Launch L{};
    bool unit = true;
    for (int j = 0; j < d; ++j) unit = unit && pr->lo[j] == 0.0 && pr->hi[j] == 1.0;
    L.kind = unit ? kStagedUnit : kStaged;
    L.fn = sample_kernel(pr->integrand, d, L.kind, f32);
    if (!L.fn) return MC_EINVAL;
    const int want = 4 * staged_waves(pr->integrand, d, f32);  // waves per CU
    L.threads = want == 24 ? 768 : 1024;
    L.window = (int)std::min<int64_t>(nb, (nb + g - 1) / g + 2);
    // as many copies as leave as many waves resident as the other launch has
    int per_cu = 0, waves = 0, others = 0;
    HIP_TRY(occupancy(out->fn, out->threads, out->lds_adj, &others));
    others *= out->threads / 64;
    const size_t fast = sizeof(double) * K * (size_t)nb;
    for (L.stage_shift = 5; L.stage_shift >= 3; --L.stage_shift) {
        L.lds_adj = lds_bytes_of(K, nb, true, f32) +
                    sizeof(double) * ns * (size_t)((f32 ? L.window : L.window + 1) + (L.window << L.stage_shift));
        if (L.lds_adj > kLdsDynamicLimit) continue;
        HIP_TRY(allow_lds(L.fn, L.lds_adj));
        HIP_TRY(occupancy(L.fn, L.threads, L.lds_adj, &per_cu));
        waves = per_cu * L.threads / 64;
        if (waves >= others && waves >= want) break;
    }
    if (L.stage_shift < 3) return MC_OK;
    // eight or more copies of every bin at as many waves do better yet (d = 6,
    // 3e7 samples, 100 bins, FP32: 149 against 164 us)
    if (out->hist_copies >= 8 && waves <= others) return MC_OK;
    mc_status st = blocks_for(L.fn, L.threads, L.lds_adj, m, 0, &L.blocks_adj);
    if (st != MC_OK) return st;
    const int64_t C = int_pow(g, K), rounds = (C + L.threads - 1) / L.threads, T = m / C * rounds;
    if (T > 0xFFFFFFFFll || rounds < 8 || T < 8 * (int64_t)L.blocks_adj) return MC_OK;
    const double filled = (double)C / (double)(rounds * L.threads);
    const double even = (double)T / L.blocks_adj / (double)((T + L.blocks_adj - 1) / L.blocks_adj);
    if (filled * even < (f32 ? 0.88 : 0.93)) return MC_OK;
    L.hist_copies = 1;
    int same = 0;
    if (L.lds_adj + fast <= kLdsDynamicLimit) {
        HIP_TRY(allow_lds(L.fn, L.lds_adj + fast));
        HIP_TRY(occupancy(L.fn, L.threads, L.lds_adj + fast, &same));
        if (same >= per_cu) {
            L.hist_copies = 2;
            L.lds_adj += fast;
        }
    }
    *out = L;
    return MC_OK;
}

mc_status geometry(const mc_problem *pr, Geometry *geo) {
    mc_status st = validate(pr);
    if (st != MC_OK) return st;
    // The calling thread's last answer, kept with everything it depends on:
    // choosing the launch takes some thirty occupancy look-ups, 4 us of a call
    // that takes 40 at 2e4 samples.
    struct Key {
        int64_t maxcalls;
        int32_t dev, integrand, dim, nbins, itmax, precision, blocks, threads, one_d, unit, spread;
        bool operator==(const Key &o) const {
            return maxcalls == o.maxcalls && dev == o.dev && integrand == o.integrand && dim == o.dim &&
                   nbins == o.nbins && itmax == o.itmax && precision == o.precision && blocks == o.blocks &&
                   threads == o.threads && one_d == o.one_d && unit == o.unit && spread == o.spread;
        }
    };
    thread_local Key kept_key{};
    thread_local Geometry kept{};
    Key key{pr->maxcalls, 0, pr->integrand, pr->dim, pr->nbins, pr->itmax, pr->precision, pr->blocks, pr->threads,
            pr->one_d, 1, 0};
    for (int j = 0; j < pr->dim; ++j)
        if (pr->lo[j] != 0.0 || pr->hi[j] != 1.0) key.unit = 0;
    // The FP64 kernels of large passes start a sample's Jacobian from the volume
    // times nb^dim (SampleArgs::j0) and multiply it by the widths, which only makes
    // it smaller.  Where that start is beyond the range of doubles, or near its
    // ends, only kernels that multiply axis by axis take the passes (kPerAxis,
    // kSplit and kFused; the traced kernel in their place: d = 8, 1e8 samples,
    // 300 bins, No-Adjust 1076 us against kPerAxis's 865).
    const double j0 = first_jacobian(pr);
    if (!is_fp32(pr) && !(j0 > 1e-200 && j0 < 1e200)) key.spread = 1;
    HIP_TRY(hipGetDevice(&key.dev));
    if (kept.total && key == kept_key) {
        *geo = kept;
        return MC_OK;
    }
    Geometry G{};
    lattice(pr->dim, pr->maxcalls, &G.g, &G.m, &G.p);
    const int d = pr->dim, nb = pr->nbins;
    const bool f32 = is_fp32(pr);
    Launch plain{};
    st = plain_launch(pr, key.spread ? kPerAxis : kPlain, G.m, &plain);
    if (st != MC_OK) return st;
    G.noadj = G.traced = plain;
    G.traced.kind = kTraced;
    G.traced.fn = sample_kernel(pr->integrand, d, kTraced, f32);
    if ((st = copies_launch(pr, G.g, G.m, G.p, plain, &G.noadj)) != MC_OK) return st;
    if (key.spread && G.noadj.kind == kCopies) G.noadj = plain;  // (kSplit multiplies axis by axis)
    G.hist_stride = (int)((d * (size_t)nb + 31) / 32 * 32);
    G.adj = G.noadj;
    if (G.noadj.kind == kCopies && G.m * G.p > kFusedMaxSamples) G.noadj = plain;
    if (!key.spread && (st = staged_launch(pr, G.g, G.m, &G.adj)) != MC_OK) return st;
    int most = 1;
    for (const Launch *L : {&G.adj, &G.noadj, &G.traced}) most = std::max({most, L->blocks_adj, L->blocks_noadj});
    const size_t most_blocks = (size_t)most;
    // The regions that mc_prepare fills, or clears for the runs to keep clear,
    // come first: the sub-cubes, the passes and the workgroups move none of
    // them, so a prepared workspace serves runs with other iteration counts.
    size_t off = 0;
    const size_t real = f32 ? sizeof(float) : sizeof(double);
    G.off_consts = off;
    off = align_up(off + real * kConstStride * d);
    G.off_grid = off;
    off = align_up(off + sizeof(double) * d * (nb + 1));
    G.off_tables = off;
    if (pr->integrand == MC_F_GAUSS_TABLES) off = align_up(off + real * (f32 ? kTablesLen32 : kTablesLen));
    // the histogram accumulators of adjusting passes and, right after them, the
    // non-finite flags, kept zero between runs
    G.off_hist = off;
    off += sizeof(double) * kHistAcc * (size_t)G.hist_stride;
    G.off_flag = off;
    off = align_up(off + kFlagBytes);
    // From here on nothing is kept from one call to the next.
    G.off_out = off;
    off = align_up(off + sizeof(double) * (4 + (size_t)d * nb));
    G.off_partials = off;
    const size_t partials = align_up(sizeof(double) * 4 * most_blocks);
    off += partials;
    // a device-steps run's state and its per-iteration (I, var)
    G.off_run = off;
    auto run_bytes = [](int itmax) { return align_up(sizeof(RunState) + sizeof(double) * 2 * (size_t)itmax); };
    G.total = off + run_bytes(pr->itmax);
    // What fused runs (see FusedArgs) need besides: a second grid, two more
    // accumulator sets and a second set of totals.  Counted whatever the iteration
    // count is, so that a workspace for more iterations holds one for fewer.
    if (d * nb <= kFusedMaxBins && pr->blocks == 0) {
        const size_t grid2 = align_up(sizeof(double) * d * (nb + 1));
        const size_t hist2 = align_up(sizeof(double) * kFusedAccs * 2 * (size_t)G.hist_stride);
        G.fusable = pr->itmax <= kFusedMaxPasses;
        G.off_fused_grid = off + run_bytes(std::min(pr->itmax, kFusedMaxPasses));
        G.off_fused_hist = G.off_fused_grid + grid2;
        G.off_fused_partials = G.off_fused_hist + hist2;
        G.total = std::max(G.total, G.off_fused_partials + partials);
    }
    kept = G;
    kept_key = key;
    *geo = G;
    return MC_OK;
}

// ------------------------------------------------------------------ one sampling pass

void fill_args(const mc_problem *pr, const Geometry &G, const Launch &L, char *ws, uint32_t iter, bool adjust,
               SampleArgs *a) {
    const double *grid = reinterpret_cast<const double *>(ws + G.off_grid);
    const void *tables = pr->integrand == MC_F_GAUSS_TABLES ? ws + G.off_tables : nullptr;
    sample_args(pr, G.g, G.m, G.p, iter, adjust, ws + G.off_consts, grid, tables, a);
    a->partials = reinterpret_cast<double *>(ws + G.off_partials);
    a->hist_acc = reinterpret_cast<double *>(ws + G.off_hist);
    a->flag = reinterpret_cast<uint32_t *>(ws + G.off_flag);
    a->stride = ((int64_t)L.blocks(adjust) * L.threads) >> L.lsplit;
    a->hist_stride = G.hist_stride;
    a->hist_copies = adjust ? L.hist_copies : 1;
    a->copy_shift = adjust ? L.copy_shift : 0;
    a->lsplit = L.lsplit;
    if (L.kind == kStaged || L.kind == kStagedUnit) {
        a->window = L.window;
        a->stage_shift = L.stage_shift;
        a->block_cubes = (uint32_t)int_pow(G.g, pr->dim - staged_slow_axes(pr->integrand, pr->dim));
        a->blocks_total = (uint32_t)(G.m / a->block_cubes);
        a->stride = L.threads;  // a round further inside a block
    }
    // the per-lane stride in base g (only d digits are used: a lane that
    // overflows the top digit has left the lattice)
    int64_t rest = a->stride;
    for (int j = 0; j < pr->dim; ++j) {
        a->sdig[j] = (int32_t)(rest % G.g);
        rest /= G.g;
    }
}

struct Events {
    hipEvent_t e[3] = {nullptr, nullptr, nullptr};
    bool ok = false;
    ~Events() {
        for (auto &x : e)
            if (x) (void)hipEventDestroy(x);
    }
    hipError_t create() {
        for (auto &x : e) {
            hipError_t err = hipEventCreate(&x);
            if (err != hipSuccess) return err;
        }
        ok = true;
        return hipSuccess;
    }
};

// Page-locked host memory, mapped for the device.
struct MappedMemory {
    static char *make(size_t bytes) {
        void *p = nullptr;
        if (hipHostMalloc(&p, bytes, hipHostMallocMapped | hipHostMallocPortable | hipHostMallocCoherent) != hipSuccess)
            return nullptr;
        std::memset(p, 0, bytes);
        return static_cast<char *>(p);
    }
    static bool free(char *p) { return hipHostFree(p) == hipSuccess; }
};

// Such memory of the calling thread (thread_local), grown on demand; a thread
// that ends leaves it to later ones.
struct Mapped {
    char *host = nullptr, *dev = nullptr;
    HeldBuffer<MappedMemory> held;
    hipError_t reserve(size_t bytes) {
        host = held.reserve(bytes);
        if (!host) return hipErrorOutOfMemory;
        void *d = nullptr;
        const hipError_t e = hipHostGetDevicePointer(&d, host, 0);
        dev = static_cast<char *>(d);
        return e;
    }
};

// Numbers of finalize launches, for the words that they write: different in
// every thread's launches, since a buffer may come from another thread; never 0,
// which fresh memory holds.
uint32_t next_seq() {
    static std::atomic<uint32_t> last{0};
    uint32_t seq = last.fetch_add(1, std::memory_order_relaxed) + 1;
    while (seq == 0) seq = last.fetch_add(1, std::memory_order_relaxed) + 1;
    return seq;
}

// Waits until *word reads seq, with a look at the stream now and then, so
// that an error or a stream that has run dry ends the wait.
hipError_t wait_word(const volatile uint32_t *word, uint32_t seq, hipStream_t s) {
    for (unsigned spin = 1; *word != seq; ++spin) {
        __builtin_ia32_pause();
        if (spin % 16384 == 0) {
            const hipError_t q = hipStreamQuery(s);
            if (q == hipSuccess && *word != seq) return hipErrorUnknown;  // drained, nothing written
            if (q != hipSuccess && q != hipErrorNotReady) return q;
        }
    }
    std::atomic_thread_fence(std::memory_order_acquire);
    return hipSuccess;
}

// One pass with the steps on the host: the grid up, sampling, finalize, and
// the result in out_host (4 + d*nb doubles).  mapped: a small kernel fetches
// the grid from page-locked memory, the finalize writes its result there and
// the host waits for the word that it writes last (allocated on first use);
// otherwise copies from and to the caller's pageable buffers, which allocate
// nothing.  The mapped form replaces two asynchronous copies and the wait on
// the stream: per pass, 1e5 samples (d = 5, FP32, 264 bins: 45 -> 39 us;
// a pass of 2e4 samples 47 -> 35, of 1e6 52 -> 46).
mc_status run_pass(const mc_problem *pr, const Geometry &G, char *ws, hipStream_t stream,
                   uint32_t iter, bool adjust, const double *h_grid, double *out_host,
                   double *trace, int64_t t0, int64_t t1, Events *ev, double *ms_sample,
                   double *ms_fin, int spin_us = 0, bool mapped = true) {
    const int d = pr->dim, nb = pr->nbins;
    const Launch &L = trace ? G.traced : G.pass(adjust);
    const int blocks = L.blocks(adjust);
    const size_t lds = L.lds(adjust);
    SampleArgs a;
    fill_args(pr, G, L, ws, iter, adjust, &a);
    a.trace = trace;
    a.t0 = t0;
    a.t1 = t1;
    const size_t grid_bytes = sizeof(double) * d * (nb + 1);
    const size_t nout = 4 + (adjust ? (size_t)d * nb : 0);
    thread_local Mapped stage;
    uint32_t seq = 0;
    double *grid_dev = reinterpret_cast<double *>(ws + G.off_grid);
    double *out_dev = reinterpret_cast<double *>(ws + G.off_out);
    uint32_t *counter = nullptr, *done = nullptr;
    const volatile uint32_t *done_host = nullptr;
    const double *out_map = nullptr;
    if (mapped) {
        // the word, the grid, the results
        const size_t o_grid = 64, o_out = o_grid + align_up(grid_bytes);
        HIP_TRY(stage.reserve(o_out + sizeof(double) * (4 + (size_t)d * nb)));
        std::memcpy(stage.host + o_grid, h_grid, grid_bytes);
        done = reinterpret_cast<uint32_t *>(stage.dev);
        done_host = reinterpret_cast<const volatile uint32_t *>(stage.host);
        out_map = reinterpret_cast<const double *>(stage.host + o_out);
        out_dev = reinterpret_cast<double *>(stage.dev + o_out);
        counter = reinterpret_cast<uint32_t *>(ws + G.off_flag + kCounterOffset);
        seq = next_seq();
        HIP_TRY(launch_upload(reinterpret_cast<const double *>(stage.dev + o_grid), grid_dev, d * (nb + 1), stream));
    } else {
        HIP_TRY(hipMemcpyAsync(grid_dev, h_grid, grid_bytes, hipMemcpyHostToDevice, stream));
    }
    if (ev) HIP_TRY(hipEventRecord(ev->e[0], stream));
    HIP_TRY(allow_lds(L.fn, lds));
    HIP_TRY(launch_sample(L.fn, blocks, L.threads, lds, stream, a));
    if (ev) HIP_TRY(hipEventRecord(ev->e[1], stream));
    HIP_TRY(launch_finalize(a.partials, a.hist_acc, blocks, d * nb, G.hist_stride, adjust ? 1 : 0, a.flag,
                            out_dev, counter, done, seq, stream));
    if (ev) HIP_TRY(hipEventRecord(ev->e[2], stream));
    if (adjust && d > 1 && !pr->one_d) AxisPool::get().prime(spin_us);
    if (mapped) {
        HIP_TRY(wait_word(done_host, seq, stream));
        std::memcpy(out_host, out_map, sizeof(double) * nout);
        if (ev) HIP_TRY(hipEventSynchronize(ev->e[2]));
    } else {
        HIP_TRY(hipMemcpyAsync(out_host, out_dev, sizeof(double) * nout, hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
    }
    if (ev) {
        float a_ms = 0.f, b_ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&a_ms, ev->e[0], ev->e[1]));
        HIP_TRY(hipEventElapsedTime(&b_ms, ev->e[1], ev->e[2]));
        *ms_sample += a_ms;
        *ms_fin += b_ms;
    }
    return out_host[2] != 0.0 ? MC_ENONFINITE : MC_OK;
}

// After a device error: what a call has queued still reads the calling thread's
// page-locked memory and the caller's tables, so it is waited for before the
// call returns the error.
mc_status drained(mc_status st, hipStream_t stream) {
    if (st == MC_EDEVICE) {
        (void)hipStreamSynchronize(stream);
        (void)hipGetLastError();
    }
    return st;
}

// Fills a workspace: constants, tables, cleared accumulators and flags, queued
// on the stream.  The constants go through page-locked memory of the calling
// thread (mapped; else pageable copies) and the tables from the caller's, so
// the stream must be waited for before either changes: with wait, here.
mc_status prepare(const mc_problem *pr, const Geometry &G, char *ws, hipStream_t stream, bool mapped, bool wait) {
    const std::vector<double> consts = axis_constants(pr);
    std::vector<float> c32, t32;
    const void *src = consts.data();
    size_t bytes = sizeof(double) * consts.size();
    if (is_fp32(pr)) {  // FP32 evaluation: every constant and table value rounded once to float
        c32.assign(consts.begin(), consts.end());
        src = c32.data();
        bytes = sizeof(float) * c32.size();  // six per axis: whole doubles
    }
    if (mapped) {
        thread_local Mapped stage;
        HIP_TRY(stage.reserve(bytes));
        std::memcpy(stage.host, src, bytes);
        HIP_TRY(launch_upload(reinterpret_cast<const double *>(stage.dev),
                              reinterpret_cast<double *>(ws + G.off_consts), (int)(bytes / sizeof(double)), stream));
    } else {
        HIP_TRY(hipMemcpyAsync(ws + G.off_consts, src, bytes, hipMemcpyHostToDevice, stream));
        wait = true;  // the copy reads this function's vectors
    }
    if (pr->integrand == MC_F_GAUSS_TABLES) {
        if (is_fp32(pr)) {
            t32.resize(kTablesLen32);
            tables_f32(pr->tables, t32.data());
            HIP_TRY(hipMemcpyAsync(ws + G.off_tables, t32.data(), sizeof(float) * kTablesLen32,
                                   hipMemcpyHostToDevice, stream));
            wait = true;
        } else {
            HIP_TRY(hipMemcpyAsync(ws + G.off_tables, pr->tables, sizeof(double) * kTablesLen,
                                   hipMemcpyHostToDevice, stream));
        }
    }
    // the histogram accumulators and the flags start at zero; whatever reads
    // them after a pass clears them again
    HIP_TRY(launch_zero(reinterpret_cast<double *>(ws + G.off_hist),
                        (G.off_flag + kFlagBytes - G.off_hist) / sizeof(double), stream));
    if (wait) HIP_TRY(hipStreamSynchronize(stream));
    return MC_OK;
}

}  // namespace

// ====================================================================== C ABI

extern "C" {

const char *mc_status_string(mc_status s) {
    switch (s) {
    case MC_OK: return "ok";
    case MC_EINVAL: return "invalid problem or argument";
    case MC_EWORKSPACE: return "workspace too small";
    case MC_ENONFINITE: return "integrand produced a non-finite value";
    case MC_EDEVICE: return "HIP device error";
    default: return "unknown status";
    }
}

mc_status mc_shape(int32_t dim, int64_t maxcalls, int64_t *g, int64_t *m, int64_t *p) {
    if (!g || !m || !p) return MC_EINVAL;
    int64_t gg, mm, pp;
    mc_status st = lattice(dim, maxcalls, &gg, &mm, &pp);
    if (st != MC_OK) return st;
    *g = gg;
    *m = mm;
    *p = pp;
    return MC_OK;
}

mc_status mc_workspace_bytes(const mc_problem *prob, size_t *bytes) {
    if (!bytes) return MC_EINVAL;
    Geometry G;
    mc_status st = geometry(prob, &G);
    if (st != MC_OK) return st;
    *bytes = G.total;
    return MC_OK;
}

mc_status mc_launch_shape(const mc_problem *prob, int32_t adjust, int32_t *blocks, int32_t *threads,
                          int32_t *lds_bytes) {
    if (!blocks || !threads || !lds_bytes) return MC_EINVAL;
    Geometry G;
    mc_status st = geometry(prob, &G);
    if (st != MC_OK) return st;
    const Launch &L = G.pass(adjust != 0);
    *blocks = L.blocks(adjust != 0);
    *threads = L.threads;
    *lds_bytes = (int32_t)L.lds(adjust != 0);
    return MC_OK;
}

mc_status mc_prepare(const mc_problem *prob, void *d_ws, size_t ws_bytes, void *stream) {
    Geometry G;
    mc_status st = geometry(prob, &G);
    if (st != MC_OK) return st;
    if (!d_ws || ws_bytes < G.total) return MC_EWORKSPACE;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    return drained(prepare(prob, G, static_cast<char *>(d_ws), s, true, true), s);
}

mc_status mc_sample_iteration(const mc_problem *prob, uint32_t iter, int32_t adjust,
                              const double *h_grid, void *d_ws, size_t ws_bytes, void *stream,
                              double *h_out, double *h_hist, void *d_trace, size_t trace_bytes,
                              int64_t t0, int64_t t1) {
    Geometry G;
    mc_status st = geometry(prob, &G);
    if (st != MC_OK) return st;
    if (!h_grid || !h_out || (!adjust && h_hist)) return MC_EINVAL;
    const int d = prob->dim, nb = prob->nbins;
    if (d_trace) {
        if (t0 < 0 || t1 < t0 || t1 > G.m) return MC_EINVAL;
        const size_t need = sizeof(double) * ((size_t)(t1 - t0) * G.p * (3 * d + 2) + 2 * (size_t)(t1 - t0));
        if (trace_bytes < need) return MC_EINVAL;
    }
    if (!d_ws || ws_bytes < G.total) return MC_EWORKSPACE;
    std::vector<double> out(4 + (size_t)d * nb);
    const hipStream_t s = static_cast<hipStream_t>(stream);
    st = drained(run_pass(prob, G, static_cast<char *>(d_ws), s, iter, adjust != 0, h_grid, out.data(),
                          static_cast<double *>(d_trace), d_trace ? t0 : 0, d_trace ? t1 : 0, nullptr, nullptr, nullptr),
                 s);
    if (st != MC_OK) return st;
    h_out[0] = out[0];
    h_out[1] = out[1];
    if (h_hist) std::copy(out.begin() + 4, out.end(), h_hist);
    return MC_OK;
}

mc_status mc_refine_grid(int32_t dim, int32_t nbins, double alpha, const double *h_hist,
                         double *h_grid) {
    if (dim < 1 || dim > MC_MAX_DIM || nbins < 2 || !(alpha > 0.0) || !h_hist || !h_grid)
        return MC_EINVAL;
    refine(dim, nbins, alpha, h_hist, h_grid);
    return MC_OK;
}

mc_status mc_refine_grid_1d(int32_t dim, int32_t nbins, double alpha, const double *h_hist,
                            double *h_grid) {
    if (dim < 1 || dim > MC_MAX_DIM || nbins < 2 || !(alpha > 0.0) || !h_hist || !h_grid)
        return MC_EINVAL;
    refine_1d(dim, nbins, alpha, h_hist, h_grid);
    return MC_OK;
}

mc_status mc_refine_grid_device(int32_t dim, int32_t nbins, double alpha, int32_t one_d,
                                const double *d_hist, double *d_grid, void *stream) {
    if (dim < 1 || dim > MC_MAX_DIM || nbins < 2 || nbins > kDeviceStepsMaxBins ||
        !(alpha > 0.0) || !std::isfinite(alpha) || (one_d != 0 && one_d != 1) || !d_hist || !d_grid)
        return MC_EINVAL;
    HIP_TRY(launch_refine(d_grid, d_hist, dim, nbins, one_d, alpha, static_cast<hipStream_t>(stream)));
    return MC_OK;
}

mc_status mc_init_grid(int32_t dim, int32_t nbins, double *h_grid) {
    if (dim < 1 || dim > MC_MAX_DIM || nbins < 2 || !h_grid) return MC_EINVAL;
    init_grid(dim, nbins, h_grid);
    return MC_OK;
}

mc_status mc_weighted_estimate(int32_t k, const double *h_I, const double *h_var, double *h_out) {
    if (k < 1 || !h_I || !h_var || !h_out) return MC_EINVAL;
    weighted(k, h_I, h_var, h_out);
    return MC_OK;
}

}  // extern "C"

namespace {

// The calling thread's host mirror of a device-steps run: its RunState, then 2 *
// itmax doubles of per-iteration results, then the grid.
hipError_t run_mirror(size_t bytes, char **host, char **dev) {
    thread_local Mapped buf;
    const hipError_t e = buf.reserve(bytes);
    *host = buf.host;
    *dev = buf.dev;
    return e;
}

// The calling thread's markers for timed device-steps runs on the current
// device, created once (and again after a change of device) and kept until
// the process ends.  Per pass two: after the sampling kernel, and "done"
// after the pass's last kernel.  Three slots each, since the next passes are
// queued before a pass is read.
struct RunEvents {
    int device = -1;
    hipEvent_t start = nullptr, sampled[3] = {}, done[3] = {};
};

hipError_t run_events(RunEvents **out) {
    thread_local RunEvents ev;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (ev.device != dev) {
        hipEvent_t *all[] = {&ev.start, &ev.sampled[0], &ev.sampled[1], &ev.sampled[2],
                             &ev.done[0], &ev.done[1], &ev.done[2]};
        for (hipEvent_t *x : all)
            if (*x) {
                (void)hipEventDestroy(*x);
                *x = nullptr;
            }
        ev.device = -1;
        for (hipEvent_t *x : all)
            if ((e = hipEventCreate(x)) != hipSuccess) return e;
        ev.device = dev;
    }
    *out = &ev;
    return hipSuccess;
}

// Alg. 2 with its steps between passes on the device: Init-Bins and the run
// state, then per pass the sampling kernel and one steps launch (totals,
// Weighted-Estimates, Check-Convergence and, while adjusting, the bin
// adjustment), all on the stream.  The sampling kernel of the next pass is
// always queued before the host waits for a pass, so the device never waits
// for the host; the steps of that pass are queued once the decision of the
// pass before is known, so a run that converges leaves only one sampling
// launch queued behind it, which does nothing.  The decisions, the
// per-iteration results and the grid come back through the mapped mirror.
mc_status integrate_device(const mc_problem *prob, const Geometry &G, char *ws, hipStream_t s,
                           mc_result *out, double *h_iters, double *h_grid, mc_timing *timing) {
    const int d = prob->dim, nb = prob->nbins, itmax = prob->itmax;
    const size_t grid_len = (size_t)d * (nb + 1);
    char *hbuf = nullptr, *dbuf = nullptr;
    HIP_TRY(run_mirror(sizeof(RunState) + sizeof(double) * (2 * (size_t)itmax + grid_len), &hbuf, &dbuf));
    RunEvents *ev = nullptr;
    if (timing) HIP_TRY(run_events(&ev));
    RunState *hm = reinterpret_cast<RunState *>(hbuf), *hm_dev = reinterpret_cast<RunState *>(dbuf);
    double *h_its = reinterpret_cast<double *>(hm + 1), *h_its_dev = reinterpret_cast<double *>(hm_dev + 1);
    double *h_gr = h_its + 2 * (size_t)itmax, *h_gr_dev = h_its_dev + 2 * (size_t)itmax;
    double *mirror_grid = h_grid ? h_gr_dev : nullptr;
    std::memset(static_cast<void *>(hm), 0, sizeof(RunState));
    hm->last = itmax - 1;
    RunState *dst = reinterpret_cast<RunState *>(ws + G.off_run);
    double *iters = reinterpret_cast<double *>(dst + 1);
    double *grid = reinterpret_cast<double *>(ws + G.off_grid);
    double *partials = reinterpret_cast<double *>(ws + G.off_partials);
    double *hist_acc = reinterpret_cast<double *>(ws + G.off_hist);
    uint32_t *flag = reinterpret_cast<uint32_t *>(ws + G.off_flag);
    hipEvent_t *done = timing ? ev->done : nullptr;
    auto pass_blocks = [&](int it) { return G.pass(it < prob->ita).blocks(it < prob->ita); };
    // the sampling kernel of pass it (and its marker)
    auto head = [&](int it) -> hipError_t {
        const bool adjust = it < prob->ita;
        const Launch &L = G.pass(adjust);
        const size_t lds = L.lds(adjust);
        SampleArgs a;
        fill_args(prob, G, L, ws, (uint32_t)it, adjust, &a);
        a.run_last = &dst->last;
        hipError_t e;
        if (timing && it == 0 && (e = hipEventRecord(ev->start, s)) != hipSuccess) return e;
        if ((e = allow_lds(L.fn, lds)) != hipSuccess) return e;
        if ((e = launch_sample(L.fn, pass_blocks(it), L.threads, lds, s, a)) != hipSuccess) return e;
        return timing ? hipEventRecord(ev->sampled[it % 3], s) : hipSuccess;
    };
    // the rest of pass it: totals, decision and bin adjustment in one launch,
    // and with timing the done marker
    auto tail = [&](int it) -> hipError_t {
        const bool adjust = it < prob->ita;
        StepsArgs sa{};
        sa.ctl = RunCtl{dst, iters, hm_dev, h_its_dev, it, itmax, prob->tau_rel, prob->chi2_max, 0};
        sa.partials = partials;
        sa.blocks = pass_blocks(it);
        sa.hist_stride = G.hist_stride;
        sa.hist_acc = hist_acc;
        sa.flag = flag;
        sa.grid = grid;
        sa.host_grid = mirror_grid;
        sa.alpha = prob->alpha;
        sa.d = d;
        sa.nb = nb;
        sa.one_d = prob->one_d;
        sa.nref = adjust ? (prob->one_d ? 1 : d) : 0;
        const hipError_t e = launch_steps(sa, s);
        if (e != hipSuccess) return e;
        return timing ? hipEventRecord(done[it % 3], s) : hipSuccess;
    };
    // until pass it's decision is in the mirror: with timing, the pass's done
    // marker; otherwise the mirror's pass count, which the steps kernel writes
    // last (no marker, which would hold the stream for a few microseconds),
    // with a look at the stream now and then, so that an error or a stream
    // that has run dry ends the wait
    auto wait_pass = [&](int it) -> hipError_t {
        if (timing) return hipEventSynchronize(done[it % 3]);
        const volatile int32_t *kk = &reinterpret_cast<volatile RunState *>(hm)->k;
        for (unsigned spin = 1;; ++spin) {
            if (*kk > it) break;
            if (spin % 1024 == 0) {
                const hipError_t q = hipStreamQuery(s);
                if (q == hipSuccess && *kk <= it) return hipErrorUnknown;  // drained, no decision
                if (q != hipSuccess && q != hipErrorNotReady) return q;
            }
        }
        std::atomic_thread_fence(std::memory_order_acquire);
        return hipSuccess;
    };
    double ms_s = 0.0, ms_f = 0.0;
    int k = 0;
    hipError_t err = launch_run_init(dst, grid, mirror_grid, d, nb, itmax, s);
    if (err == hipSuccess) err = head(0);
    if (err == hipSuccess) err = tail(0);
    if (err == hipSuccess && itmax > 1) err = head(1);
    for (int it = 0; err == hipSuccess && it < itmax; ++it) {
        if ((err = wait_pass(it)) != hipSuccess) break;
        k = it + 1;
        if (timing) {
            float a_ms = 0.f, b_ms = 0.f;
            hipEvent_t from = it == 0 ? ev->start : done[(it - 1) % 3];
            if ((err = hipEventElapsedTime(&a_ms, from, ev->sampled[it % 3])) != hipSuccess ||
                (err = hipEventElapsedTime(&b_ms, ev->sampled[it % 3], done[it % 3])) != hipSuccess)
                break;
            ms_s += a_ms;
            ms_f += b_ms;
        }
        if (reinterpret_cast<volatile RunState *>(hm)->last <= it) break;  // pass it ended the run
        // the run goes on: the rest of pass it + 1, whose sampling kernel is
        // running, and the sampling kernel after it
        if ((err = tail(it + 1)) != hipSuccess) break;
        if (it + 2 < itmax && (err = head(it + 2)) != hipSuccess) break;
    }
    // a sampling launch queued after the last pass does nothing; wait for it too
    const hipError_t err2 = hipStreamSynchronize(s);
    HIP_TRY(err);
    HIP_TRY(err2);
    const volatile RunState *v = hm;
    if (v->status == kRunNonFinite) return MC_ENONFINITE;
    if (h_grid) std::memcpy(h_grid, h_gr, sizeof(double) * grid_len);
    out->estimate = v->est[0];
    out->error = v->est[1];
    out->chi2_dof = v->est[2];
    out->iterations = k;
    out->converged = v->status == kRunConverged ? 1 : 0;
    out->calls = (int64_t)k * G.m * G.p;
    if (h_iters)
        for (int i = 0; i < k; ++i) {
            h_iters[2 * i] = h_its[i];
            h_iters[2 * i + 1] = h_its[itmax + i];
        }
    if (timing) {
        timing->sample_ms = ms_s;
        timing->finalize_ms = ms_f;
        timing->launches = k;
        const Launch &L = G.pass(prob->ita > 0);
        timing->blocks = L.blocks(prob->ita > 0);
        timing->threads = L.threads;
        timing->lds_bytes = (int32_t)L.lds(prob->ita > 0);
    }
    return MC_OK;
}

// Whether the steps of a device-steps run go into the sampling launches
// themselves (FusedArgs), and the launch with the LDS they need.
bool fused_launch(const mc_problem *prob, const Geometry &G, Launch *out) {
    if (!G.fusable || (G.noadj.kind != kCopies && G.noadj.kind != kSplit) || G.m * G.p > kFusedMaxSamples)
        return false;
    // A run to a target may end after two passes, and then pays the steps of
    // every axis in every workgroup three times
    if (prob->tau_rel > 0.0 && prob->dim * prob->nbins > kFusedTargetBins) return false;
    Launch L = G.noadj;  // (passes this small are never staged)
    L.kind = kFused;
    L.fn = sample_kernel(prob->integrand, prob->dim, kFused, is_fp32(prob));
    if (!L.fn) return false;
    // each workgroup adjusts every axis: with 256 threads those of three axes
    // of 100 bins take 20.0 us per pass, with 512 17.1
    if (!prob->threads && L.threads == 256 && prob->dim * prob->nbins > 256) {
        L.threads = 512;
        L.blocks_adj = L.blocks_noadj = (int)std::max<int64_t>(1, ((G.m << L.lsplit) + 511) / 512);
    }
    const size_t need = lds_bytes_of(prob->dim, prob->nbins, false, is_fp32(prob)) +
                        sizeof(double) * fused_scratch(prob->dim, prob->nbins);
    if (need > kLdsDynamicLimit) return false;
    int cus = 0;
    if (compute_units(&cus) != hipSuccess) return false;
    for (int adj = 0; adj < 2; ++adj) {
        size_t &lds = adj ? L.lds_adj : L.lds_noadj;
        int &blocks = adj ? L.blocks_adj : L.blocks_noadj;
        lds = std::max(lds, need);
        int per_cu = 0;
        if (allow_lds(L.fn, lds) != hipSuccess || occupancy(L.fn, L.threads, lds, &per_cu) != hipSuccess || per_cu < 1)
            return false;
        blocks = std::min(blocks, per_cu * cus);
    }
    *out = L;
    return true;
}

// A fused run: pass n's launch does the steps that follow pass n - 1 and then
// samples; one steps launch follows the last pass.  Without a target the whole
// run is queued at once; with one, kAhead launches ahead of the last
// decision seen in the mirror (a run that ends leaves that many launches
// queued, which return at once).
mc_status integrate_fused(const mc_problem *prob, const Geometry &G, const Launch &L, char *ws, hipStream_t s,
                          mc_result *out, double *h_iters, double *h_grid) {
    constexpr int kAhead = 2;
    const int d = prob->dim, nb = prob->nbins, itmax = prob->itmax;
    const size_t grid_len = (size_t)d * (nb + 1);
    char *hbuf = nullptr, *dbuf = nullptr;
    HIP_TRY(run_mirror(sizeof(RunState) + sizeof(double) * (2 * (size_t)itmax + grid_len), &hbuf, &dbuf));
    RunState *hm = reinterpret_cast<RunState *>(hbuf), *hm_dev = reinterpret_cast<RunState *>(dbuf);
    double *h_its = reinterpret_cast<double *>(hm + 1), *h_its_dev = reinterpret_cast<double *>(hm_dev + 1);
    double *h_gr = h_its + 2 * (size_t)itmax, *h_gr_dev = h_its_dev + 2 * (size_t)itmax;
    std::memset(static_cast<void *>(hm), 0, sizeof(RunState));
    RunState *dst = reinterpret_cast<RunState *>(ws + G.off_run);
    double *iters = reinterpret_cast<double *>(dst + 1);
    auto dbl = [&](size_t off) { return reinterpret_cast<double *>(ws + off); };
    auto u32 = [&](size_t off) { return reinterpret_cast<uint32_t *>(ws + off); };
    // the grid of pass n is version min(n, ita)
    auto version = [&](int n) { return std::min(n, prob->ita); };
    SampleArgs a[2];
    for (int adj = 0; adj < 2; ++adj) {
        if (adj ? prob->ita > 0 : prob->ita < itmax) fill_args(prob, G, L, ws, 0, adj != 0, &a[adj]);
    }
    auto pass = [&](int n) -> hipError_t {
        const bool adjust = n < prob->ita;
        SampleArgs &p = a[adjust ? 1 : 0];
        p.iter = (uint32_t)n;
        p.grid = dbl(G.grid_set(version(n > 0 ? n - 1 : 0)));
        p.partials = dbl(G.partials_set(n));
        p.hist_acc = dbl(G.hist_set(n));
        p.flag = u32(G.flag_set(n));
        FusedArgs &z = p.fused;
        z.refine = n > 0 && n - 1 < prob->ita ? 1 : 0;
        z.prev_blocks = n > 0 ? L.blocks(n - 1 < prob->ita) : 0;
        z.itmax = itmax;
        z.prev_partials = dbl(G.partials_set(n + 1));
        z.prev_acc = dbl(G.hist_set(n + 2));
        z.clear_acc = dbl(G.hist_set(n + 1));
        z.prev_flag = u32(G.flag_set(n + 2));
        z.clear_flag = u32(G.flag_set(n + 1));
        z.next_grid = dbl(G.grid_set(version(n)));
        z.state = dst;
        z.iters = iters;
        z.host = hm_dev;
        z.host_iters = h_its_dev;
        z.host_grid = h_grid ? h_gr_dev : nullptr;
        z.tau_rel = prob->tau_rel;
        z.chi2_max = prob->chi2_max;
        z.alpha = prob->alpha;
        return launch_sample(L.fn, L.blocks(adjust), L.threads, L.lds(adjust), s, p);
    };
    auto last = [&]() -> hipError_t {
        const bool adjust = itmax - 1 < prob->ita;
        StepsArgs sa{};
        sa.ctl = RunCtl{dst, iters, hm_dev, h_its_dev, itmax - 1, itmax, prob->tau_rel, prob->chi2_max, 1};
        sa.partials = dbl(G.partials_set(itmax - 1));
        sa.blocks = L.blocks(adjust);
        sa.hist_stride = G.hist_stride;
        sa.hist_acc = dbl(G.hist_set(itmax - 1));
        sa.flag = u32(G.flag_set(itmax - 1));
        sa.grid = dbl(G.grid_set(version(itmax - 1)));
        sa.host_grid = h_grid ? h_gr_dev : nullptr;
        sa.alpha = prob->alpha;
        sa.d = d;
        sa.nb = nb;
        sa.one_d = prob->one_d;
        sa.nref = adjust ? (prob->one_d ? 1 : d) : 0;
        sa.clear_acc = dbl(G.hist_set(itmax + 1));  // pass itmax - 2's
        sa.clear_flag = u32(G.flag_set(itmax + 1));
        return launch_steps(sa, s);
    };
    HIP_TRY(allow_lds(L.fn, std::max(L.lds_adj, L.lds_noadj)));
    const volatile RunState *v = hm;
    hipError_t err = hipSuccess;
    for (int n = 0; n <= itmax && err == hipSuccess && v->status == kRunGoing; ++n) {
        err = n < itmax ? pass(n) : last();
        if (!(prob->tau_rel > 0.0)) continue;
        for (unsigned spin = 1; err == hipSuccess && n - v->k >= kAhead && v->status == kRunGoing; ++spin)
            if (spin % 1024 == 0) {
                const hipError_t q = hipStreamQuery(s);
                if (q == hipSuccess && n - v->k >= kAhead && v->status == kRunGoing) err = hipErrorUnknown;
                if (q != hipSuccess && q != hipErrorNotReady) err = q;
            }
    }
    const hipError_t err2 = hipStreamSynchronize(s);
    HIP_TRY(err);
    HIP_TRY(err2);
    if (v->status == kRunNonFinite) return MC_ENONFINITE;
    const int k = v->k;
    if (h_grid) std::memcpy(h_grid, h_gr, sizeof(double) * grid_len);
    out->estimate = v->est[0];
    out->error = v->est[1];
    out->chi2_dof = v->est[2];
    out->iterations = k;
    out->converged = v->status == kRunConverged ? 1 : 0;
    out->calls = (int64_t)k * G.m * G.p;
    if (h_iters)
        for (int i = 0; i < k; ++i) {
            h_iters[2 * i] = h_its[i];
            h_iters[2 * i + 1] = h_its[itmax + i];
        }
    return MC_OK;
}

// Whether a run keeps the steps between passes on the device: asked for, and
// the bin adjustment's LDS holds nb.
bool steps_on_device(const mc_problem *prob) {
    return prob->device_steps == 1 && prob->nbins <= kDeviceStepsMaxBins;
}

// Alg. 2 on a workspace; upload: copy the constants and tables first
// (otherwise a previous mc_prepare() of the same problem left them there).
mc_status integrate_on(const mc_problem *prob, const Geometry &G, char *ws, hipStream_t s, bool upload,
                       mc_result *out, double *h_iters, double *h_grid, mc_timing *timing, bool pinned) {
    mc_status st;
    if (upload) {
        // (the passes that follow on the stream are waited for before this returns)
        st = prepare(prob, G, ws, s, pinned, false);
        if (st != MC_OK) return st;
    }
    if (pinned && steps_on_device(prob)) {
        // with timing the passes and the steps stay launches of their own
        Launch L;
        if (!timing && fused_launch(prob, G, &L)) return integrate_fused(prob, G, L, ws, s, out, h_iters, h_grid);
        return integrate_device(prob, G, ws, s, out, h_iters, h_grid, timing);
    }

    const int d = prob->dim, nb = prob->nbins;
    std::vector<double> grid((size_t)d * (nb + 1)), buf(4 + (size_t)d * nb);
    std::vector<double> Is(prob->itmax), Vs(prob->itmax);
    init_grid(d, nb, grid.data());
    Events ev;
    if (timing) HIP_TRY(ev.create());
    double ms_s = 0.0, ms_f = 0.0, est[3] = {0.0, 0.0, NAN};
    int k = 0, converged = 0;
    int spin_us = 0;  // how long primed refinement threads spin: about one pass
    for (int it = 0; it < prob->itmax; ++it) {
        const bool adjust = it < prob->ita;
        const auto pass_start = std::chrono::steady_clock::now();
        st = run_pass(prob, G, ws, s, (uint32_t)it, adjust, grid.data(), buf.data(), nullptr, 0, 0,
                      timing ? &ev : nullptr, &ms_s, &ms_f, spin_us, pinned);
        if (st != MC_OK) return st;
        const double pass_us = std::chrono::duration<double, std::micro>(
                                   std::chrono::steady_clock::now() - pass_start).count();
        spin_us = (int)std::min(2.0 * pass_us + 200.0, 20000.0);
        Is[it] = buf[0];
        Vs[it] = buf[1];
        k = it + 1;
        weighted(k, Is.data(), Vs.data(), est);
        if (adjust) {
            if (prob->one_d)
                refine_1d(d, nb, prob->alpha, buf.data() + 4, grid.data());
            else
                refine(d, nb, prob->alpha, buf.data() + 4, grid.data());
        }
        if (check_convergence(prob, k, est)) {
            converged = 1;
            break;
        }
    }
    out->estimate = est[0];
    out->error = est[1];
    out->chi2_dof = est[2];
    out->iterations = k;
    out->converged = converged;
    out->calls = (int64_t)k * G.m * G.p;
    if (h_iters)
        for (int i = 0; i < k; ++i) {
            h_iters[2 * i] = Is[i];
            h_iters[2 * i + 1] = Vs[i];
        }
    if (h_grid) std::copy(grid.begin(), grid.end(), h_grid);
    if (timing) {
        timing->sample_ms = ms_s;
        timing->finalize_ms = ms_f;
        timing->launches = k;
        const Launch &L = G.pass(prob->ita > 0);
        timing->blocks = L.blocks(prob->ita > 0);
        timing->threads = L.threads;
        timing->lds_bytes = (int32_t)L.lds(prob->ita > 0);
    }
    return MC_OK;
}

mc_status integrate(const mc_problem *prob, void *d_ws, size_t ws_bytes, void *stream, bool upload,
                    mc_result *out, double *h_iters, double *h_grid, mc_timing *timing,
                    bool pinned = true) {
    if (!out) return MC_EINVAL;
    Geometry G;
    const mc_status st = geometry(prob, &G);
    if (st != MC_OK) return st;
    if (!d_ws || ws_bytes < G.total) return MC_EWORKSPACE;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    return drained(integrate_on(prob, G, static_cast<char *>(d_ws), s, upload, out, h_iters, h_grid, timing, pinned), s);
}

}  // namespace

extern "C" {

mc_status mc_integrate(const mc_problem *prob, void *d_ws, size_t ws_bytes, void *stream,
                       mc_result *out, double *h_iters, double *h_grid, mc_timing *timing) {
    return integrate(prob, d_ws, ws_bytes, stream, true, out, h_iters, h_grid, timing);
}

mc_status mc_integrate_prepared(const mc_problem *prob, void *d_ws, size_t ws_bytes, void *stream,
                                mc_result *out, double *h_iters, double *h_grid,
                                mc_timing *timing) {
    return integrate(prob, d_ws, ws_bytes, stream, false, out, h_iters, h_grid, timing);
}

int32_t mcubes_launch_kind(const mc_problem *prob, int32_t adjust, int32_t run) {
    Geometry G;
    Launch L;
    if (geometry(prob, &G) != MC_OK) return -1;
    if (run && steps_on_device(prob) && fused_launch(prob, G, &L)) return L.kind;
    return G.pass(adjust != 0).kind;
}

}  // extern "C"

namespace mcubes {
namespace host {

mc_status integrate_unpinned(const mc_problem *prob, void *d_ws, size_t ws_bytes, void *stream,
                             mc_result *out, double *h_iters, double *h_grid) {
    return integrate(prob, d_ws, ws_bytes, stream, true, out, h_iters, h_grid, nullptr, false);
}

}  // namespace host
}  // namespace mcubes
