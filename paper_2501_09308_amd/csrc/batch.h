// Device-side tables of the batched serving step.
#pragma once

#include <hip/hip_runtime.h>

#include "dense_tile.h"
#include "xrdvi_device.h"

namespace xrdvi {

constexpr int kMaxSlots = 512;

// Kernel kinds of one batched step, each with its own work prefix.  The
// fused tile and the peak-major adjoint have one kernel per variant
// (windowed or dense, symmetric or asymmetric peaks, constant or sec-law
// width), so that each kernel keeps the register budget of its
// single-analysis counterpart.
enum BatchKind { kSample = 0, kWindows, kWindowsSec, kCand,
                 kFusedWin, kFusedDense, kFusedWinAsym, kFusedDenseAsym,
                 kFusedWinSec, kFusedDenseSec, kFusedWinAsymSec,
                 kFusedDenseAsymSec,
                 kAdjoint, kAdjointAsym, kAdjointSec, kAdjointAsymSec,
                 kElbo, kGrad, kKinds };

constexpr int fused_kind(bool win, bool asym, bool sec) {
    return kFusedWin + (win ? 0 : 1) + (asym ? 2 : 0) + (sec ? 4 : 0);
}
constexpr int adjoint_kind(bool asym, bool sec) {
    return kAdjoint + (asym ? 1 : 0) + (sec ? 2 : 0);
}

// Fixed persistent grids (blocks) of the batched kernels; block b takes units
// b, b + grid, ...  The windowed forward and adjoint have several times the
// blocks that fit the chip (1792 and 2048): their units differ in length,
// and blocks that start as others end even that out, where a grid a little
// over what fits runs its last blocks almost alone (with 1536 fitting, eight analyses of N
// 2000-12000, K 20-300, S 32: forward 166 us a step with 2048 blocks, 149 with
// 3072, 145 with 6144, 141 with 8192; adjoint 160 with 2048, 148 with 8192,
// 143 with 16384).  Blocks left without a unit end at once: a single analysis
// of 8 phases takes 46 us a step with either.  The dense kernel's LDS leaves
// one block of four samples per CU, so 256 (eight analyses of N 1500-5000, K
// 10-80, S 32, 60 steps: 14.0 ms, with 2048 blocks 14.6); of its blocks of one
// sample two share a CU, and it has twice as many.
constexpr int kGridSmall = 1024;
constexpr int kGridLarge = 2048;
constexpr int kGridWin = 8192;
constexpr int kGridAdjoint = 16384;
constexpr int kGridDense = 256;
constexpr int kGridElbo = 256;

// One resident analysis: its problem, per-step state and optimiser state.
struct SlotDev {
    ProbDev P;
    StepDev st;
    double *loc, *logscale;                      // [D K] variational params
    double *m1_loc, *m2_loc, *m1_ls, *m2_ls;     // [D K] Adam moments
    double *trace;                               // [steps] ELBO per step
    int *step;                                   // steps done so far
    int steps;
    uint64_t seed;
    double lr;
};

// Membership of the next batched step: resident slot ids and, per kernel
// kind, the prefix of work units over them.
struct SchedDev {
    int n;
    int slot[kMaxSlots];
    int pre[kKinds][kMaxSlots + 1];
};

// Work units of each kind for one analysis.
inline void batch_units(const ProbDev &P, int S, int units[kKinds]) {
    const bool win = P.cutoff > 0.0, asym = P.D == 5, sec = P.sec != 0;
    const long long nkb = (P.K + kWave - 1) / kWave;
    for (int k = 0; k < kKinds; ++k) units[k] = 0;
    units[kSample] = (int)(S * nkb);
    if (win || sec)
        units[sec ? kWindowsSec : kWindows] = (int)(((long long)S * P.T + 255) / 256);
    if (win && !sec) {   // the forward's candidates, found once per step
        // the phases' extremes over the samples, 64 phases per unit, run as
        // the window step's first units
        units[kWindows] += (int)nkb;
        units[kCand] = (int)(((long long)P.K + kCandThreads - 1) / kCandThreads) * P.ntiles;
    }
    const DenseCut cut = dense_cut(P.N, S);
    units[fused_kind(win, asym, sec)] = win ? P.ntiles * S : cut.tiles(P.N) * cut.groups(S);
    // (the windowed adjoint's last unit is the ELBO)
    if (win) units[adjoint_kind(asym, sec)] = P.K * S + 1;
    else units[kElbo] = 1;
    units[kGrad] = win ? (P.K + kWaves - 1) / kWaves : P.K;   // windowed: a phase per wave
}

// Variant class of an analysis (0..7): windowed (bit 0), asymmetric peaks
// (bit 1), sec-law width (bit 2).  Each class has its own fused and adjoint
// kernels; a batched step launches only those of the resident classes.
inline int batch_class(const ProbDev &P) {
    return (P.cutoff > 0.0 ? 1 : 0) | (P.D == 5 ? 2 : 0) | (P.sec != 0 ? 4 : 0);
}

// Bits of the sets of resident classes beside bit c for class c: some dense
// analysis has one, or four, samples per block (a kernel each).
constexpr unsigned kDenseOne = 1u << 8, kDenseFour = 1u << 9;
constexpr int kClassSets = 1 << 10;
inline unsigned class_bits(const ProbDev &P, int S) {
    const unsigned c = 1u << batch_class(P);
    if (P.cutoff > 0.0) return c;
    return c | (dense_cut(P.N, S).group == 1 ? kDenseOne : kDenseFour);
}

// One batched step over the resident analyses, whose class_bits are set in
// `classes`.
hipError_t launch_batch_step(const SlotDev *tab, const SchedDev *sch,
                             hipStream_t stream, unsigned classes);

// Enters an analysis into the slot table: its entry, step 0, a zero trace.
hipError_t launch_enter_slot(const SlotDev &d, SlotDev *entry, hipStream_t stream);

}  // namespace xrdvi
