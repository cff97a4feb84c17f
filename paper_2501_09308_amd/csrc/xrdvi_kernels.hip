// Global kernels of one analysis step (gfx950).  See xrdvi_device.h for the
// per-tile work and the data layout.
#include <type_traits>

#include "dense_tile.h"
#include "xrdvi_device.h"
#include "xrdvi_internal.h"
#include "xrdvi_steps.h"

namespace xrdvi {

// Problem preparation: ln y!, tile-relative FP32 grid and peak positions.
__global__ void k_prepare_points(ProbDev P, double *lgy, float *u, float *ul) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P.ntiles * kTile) return;
    const double xref = P.x[min(i / P.ref * P.ref + P.ref / 2, P.N - 1)];
    if (i < P.N) {
        lgy[i] = lgamma(P.y[i] + 1.0);
        const double v = P.x[i] - xref;
        const float vh = (float)v;
        u[i] = vh;
        ul[i] = (float)(v - (double)vh);
    } else {
        u[i] = 0.f;
        ul[i] = 0.f;
    }
}

// Position index of each phase (see ProbDev::ptab), a thread per entry.
__global__ void k_prepare_index(ProbDev P, int *ptab) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P.K * (kTabBuckets + 1)) return;
    const int k = i / (kTabBuckets + 1), b = i % (kTabBuckets + 1);
    const double v = P.tab_inv > 0.0 ? P.tab_x0 + b / P.tab_inv : P.tab_x0;
    int lo = P.off[k], hi = P.off[k + 1];
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (P.pos[mid] < v) lo = mid + 1; else hi = mid;
    }
    ptab[i] = lo;
}

__global__ void k_prepare_peaks(ProbDev P, float *pt, float *ptl) {
    const int t = blockIdx.y;
    const double xref = P.x[min(t * P.ref + P.ref / 2, P.N - 1)];
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < P.T;
         j += gridDim.x * blockDim.x) {
        const double v = P.pos[j] - xref;
        const float vh = (float)v;
        pt[(size_t)t * P.T + j] = vh;
        ptl[(size_t)t * P.T + j] = (float)(v - (double)vh);
    }
}

// The near ranges of a dense problem, one thread per (kind of tile, margin,
// tile, phase).
__global__ __launch_bounds__(64) void k_prepare_near(ProbDev P, int2 *near) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x, t = blockIdx.y;
    const int kind = blockIdx.z / P.near_levels, level = blockIdx.z % P.near_levels;
    if (k < P.K && t < (int)near_tiles(P.N, kind))
        near[near_offset(P.N, P.K, P.near_levels, kind, level) + (size_t)t * P.K + k] =
            dense_near_entry(P, kind ? 4 : 2, level, t, k);
}

// a1: grid (ceil(K/64), S), 256 threads.
__global__ __launch_bounds__(256) void k_sample(
    ProbDev P, StepDev st, const double *__restrict__ loc,
    const double *__restrict__ logscale, const double *__restrict__ eps_in,
    uint64_t seed, uint64_t step) {
    __shared__ SampleSmem sm;
    sample_block(P, st, loc, logscale, eps_in, seed, step, blockIdx.y,
                 blockIdx.x, gridDim.x, sm);
}

// Constants of given constrained samples (profile entry).
__global__ void k_phi_consts(ProbDev P, int S, const double *__restrict__ phi,
                             float4 *pk, float *pkr) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    const int s = blockIdx.y;
    if (k >= P.K || s >= S) return;
    const double *ph = phi + (size_t)s * P.D * P.K;
    const size_t o = (size_t)s * P.K + k;
    if (P.D == 5) {
        const double al = ph[4 * P.K + k];
        pk[o] = phase_consts(ph[k], ph[P.K + k], ph[2 * P.K + k],
                             ph[3 * P.K + k], asym_norm(al));
        pkr[o] = asym_iw2(ph[2 * P.K + k], al);
    } else {
        pk[o] = phase_consts(ph[k], ph[P.K + k], ph[2 * P.K + k],
                             ph[3 * P.K + k]);
    }
}

// a2: one thread per (sample, peak).  perm != NULL writes the caller's
// peak order; psec != NULL also writes the sec-law peak records.
template <bool SEC>
__global__ __launch_bounds__(256) void k_windows(ProbDev P, int S, const double *__restrict__ phi,
                          int *lo, int *hi, const int *__restrict__ perm,
                          float4 *psec) {
    const size_t n = (size_t)S * P.T;
    for (size_t g = (size_t)blockIdx.x * 256; g < n; g += (size_t)gridDim.x * 256)
        windows_elem<SEC>(P, S, phi, lo, hi, perm, g, psec);
}

// a2 (windowed, constant width): the window step and the phases' extremes
// over the samples in one launch.  Blocks [0, next) take 64 phases each,
// the others one thread per (sample, peak) as k_windows.
__global__ __launch_bounds__(kCandThreads) void k_windows_ext(ProbDev P, StepDev st,
                                                              const double *__restrict__ phi,
                                                              int next) {
    __shared__ CandExtSmem sm;
    if ((int)blockIdx.x < next) {
        cand_ext_block(P, st, phi, blockIdx.x * kWave, sm);
        return;
    }
    const size_t n = (size_t)st.S * P.T;
    const size_t nb = gridDim.x - next;
    for (size_t g = (size_t)(blockIdx.x - next) * 256; g < n; g += nb * 256)
        windows_elem<false>(P, st.S, phi, st.lo, st.hi, nullptr, g, nullptr);
}

// The candidate ranges, grid (ceil(K / 256), ntiles), one thread per
// (tile, phase).
__global__ __launch_bounds__(kCandThreads) void k_cand(ProbDev P, StepDev st) {
    const int k = blockIdx.x * kCandThreads + threadIdx.x;
    if (k < P.K) cand_elem(P, st, blockIdx.y, k);
}

// a3 + a4 (+ a6), dense: one (tile, group of SG samples) per block, grid
// (tiles, groups), blocks ordered by XCD (the samples of a tile share its
// positions and counts in one L2, and their adjoint partials, adjacent in
// memory, merge there before write-back).  Four waves per SIMD (128 VGPRs), with
// one sample per block eight, so that two blocks hide each other's latencies
// (35 x 28, N = 1000, S = 60, 480 blocks: 46.7 us, one block at a time 55.7).
template <bool GRAD, bool ASYM, bool SEC, int SG, int LV, bool CUT>
__global__ __launch_bounds__(kDenseWaves * kWave, SG == 1 ? 8 : 4) void k_dense(ProbDev P, StepDev st,
                                                                  float *f_out, int wide) {
    if constexpr (LV == 4) {
        // the wide tiles first, then those of two leaves (see dense_cut)
        __shared__ union {
            DenseSmem<kDenseWaves, SG, 4, ASYM, SEC> wide;
            DenseSmem<kDenseWaves, SG, 2, ASYM, SEC> two;
        } sm;
        const int ng = (st.S + SG - 1) / SG, b = blockIdx.x + blockIdx.y * gridDim.x;
        if (b < wide * ng) {
            const int2 tg = xcd_tile_sample(b, wide, ng);
            dense_tile<GRAD, ASYM, SEC, kDenseWaves, SG, 4, CUT>(P, st, tg.x, tg.x, tg.y, f_out,
                                                            sm.wide);
        } else {
            const int2 tg = xcd_tile_sample(b - wide * ng, st.nt - wide, ng);
            dense_tile<GRAD, ASYM, SEC, kDenseWaves, SG, 2, CUT>(P, st, 2 * wide + tg.x,
                                                            wide + tg.x, tg.y, f_out, sm.two);
        }
    } else {
        __shared__ DenseSmem<kDenseWaves, SG, LV, ASYM, SEC> sm;
        const int2 tg = xcd_tile_sample(st.nt, (st.S + SG - 1) / SG);
        dense_tile<GRAD, ASYM, SEC, kDenseWaves, SG, LV, CUT>(P, st, tg.x, tg.x, tg.y, f_out, sm);
    }
}

// ... of few peaks (see dense_direct); two blocks share a CU.
template <bool GRAD, bool ASYM, bool SEC, int SG, int LV>
__global__ __launch_bounds__(kDenseWaves * kWave, 8) void k_direct(ProbDev P, StepDev st,
                                                                   float *f_out, int wide) {
    __shared__ union {
        DirectSmem<kDenseWaves, SG, LV, ASYM> wide;
        DirectSmem<kDenseWaves, SG, 2, ASYM> two;
    } sm;
    const int ng = (st.S + SG - 1) / SG, b = blockIdx.x + blockIdx.y * gridDim.x;
    if (LV == 2 || b < wide * ng) {
        const int2 tg = xcd_tile_sample(b, LV == 2 ? st.nt : wide, ng);
        dense_direct<GRAD, ASYM, SEC, kDenseWaves, SG, LV>(P, st, tg.x, tg.x, tg.y, f_out,
                                                           sm.wide);
    } else {
        const int2 tg = xcd_tile_sample(b - wide * ng, st.nt - wide, ng);
        dense_direct<GRAD, ASYM, SEC, kDenseWaves, SG, 2>(P, st, 2 * wide + tg.x, wide + tg.x,
                                                          tg.y, f_out, sm.two);
    }
}

// a3 + a4 (windowed): forward tile over its staged peak records; grid
// (ntiles, S), kBlock threads, blocks ordered by XCD.  The register budget is
// held to the occupancy the staging space allows (seven blocks per CU, six
// with asymmetric records or the sec law).
template <bool ASYM, bool SEC, bool UNIF>
__global__ __launch_bounds__(kBlock, ASYM || SEC ? 6 : 7) void k_win(ProbDev P, StepDev st,
                                                float *f_out) {
    __shared__ WinSmem<ASYM> sm;
    const int2 ts = st.S % kXcds == 0 ? xcd_sample_group(st.S)
                                      : xcd_tile_sample(P.ntiles, st.S);
    win_tile<ASYM, SEC, UNIF>(P, st, ts.x, ts.y, f_out, sm);
}

// a6 (windowed): peak-major adjoint, one block per (sample, phase), and a5 by
// the first block; grid (K, S + 1), kBlock threads.
template <bool ASYM, bool SEC, int LN>
__global__ __launch_bounds__(kBlock) void k_adjoint_win(ProbDev P, StepDev st, ElboOut out) {
    __shared__ double red[kWaves][12];
    if (blockIdx.y == 0) {
        __shared__ ElboSmem<kBlock> sm;
        if (blockIdx.x > 0 || !out.logscale) return;
        const double e = elbo_block<kBlock>(P, st, out.logscale, out.loglik, sm, out.logp);
        if (threadIdx.x == 0 && out.elbo) *out.elbo = e;
        return;
    }
    adjoint_phase<ASYM, SEC, LN>(P, st, blockIdx.y - 1, blockIdx.x, red);
}

// a5: one block of NT threads (see elbo_block).
template <int NT>
__global__ __launch_bounds__(NT) void k_elbo(ProbDev P, StepDev st, ElboOut out) {
    __shared__ ElboSmem<NT> sm;
    const double e = elbo_block<NT>(P, st, out.logscale, out.loglik, sm, out.logp);
    if (threadIdx.x == 0 && out.elbo) *out.elbo = e;
}

// a7: one block of 256 threads per phase.
__global__ __launch_bounds__(256) void k_grad(ProbDev P, StepDev st,
                                              double scale,
                                              const double *scale_dev,
                                              double *gloc,
                                              double *glogscale,
                                              double *gz_out) {
    __shared__ GradSmem sm;
    grad_block(P, st, blockIdx.x, scale, scale_dev, gloc, glogscale, nullptr,
               nullptr, nullptr, sm, gz_out);
}

// a7, windowed: one wave per phase, grid ceil(K / 4).
__global__ __launch_bounds__(256) void k_grad_win(ProbDev P, StepDev st,
                                                  double scale,
                                                  const double *scale_dev,
                                                  double *gloc,
                                                  double *glogscale,
                                                  double *gz_out) {
    const int k = blockIdx.x * kWaves + (int)(threadIdx.x / kWave);
    if (k < P.K)
        grad_wave(P, st, k, scale, scale_dev, gloc, glogscale, nullptr, nullptr,
                  nullptr, gz_out);
}

// a8: Adam ascent step on n coordinates.
__global__ void k_adam(int n, double *theta, double *m1, double *m2,
                       const double *__restrict__ g, int t, double lr,
                       double b1, double b2, double eps) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) adam_update(theta[j], m1[j], m2[j], g[j], t, lr, b1, b2, eps);
}

// ---- launchers ------------------------------------------------------------

hipError_t launch_prepare(const ProbDev &P, double *lgy, float *u, float *ul,
                          int *ptab, float *pt, float *ptl, int2 *near,
                          hipStream_t stream) {
    const int np = P.ntiles * kTile;
    k_prepare_points<<<(np + 255) / 256, 256, 0, stream>>>(P, lgy, u, ul);
    k_prepare_index<<<(P.K * (kTabBuckets + 1) + 255) / 256, 256, 0, stream>>>(P, ptab);
    if (P.T > 0) {
        dim3 g((P.T + 255) / 256 < 64 ? (P.T + 255) / 256 : 64, (P.N + P.ref - 1) / P.ref);
        k_prepare_peaks<<<g, 256, 0, stream>>>(P, pt, ptl);
    }
    if (P.cutoff == 0.0 && !P.sec) {
        dim3 g((P.K + 63) / 64, (unsigned)near_tiles(P.N, 0), P.near_kinds * P.near_levels);
        k_prepare_near<<<g, 64, 0, stream>>>(P, near);
    }
    return hipGetLastError();
}

hipError_t launch_sample(const ProbDev &P, const StepDev &st,
                         const double *loc, const double *logscale,
                         const double *eps, uint64_t seed, uint64_t step,
                         hipStream_t stream) {
    dim3 g((P.K + kWave - 1) / kWave, st.S);
    k_sample<<<g, 256, 0, stream>>>(P, st, loc, logscale, eps, seed, step);
    return hipGetLastError();
}

hipError_t launch_phi_consts(const ProbDev &P, int S, const double *phi,
                             float4 *pk, float *pkr, hipStream_t stream) {
    dim3 g((P.K + kWave - 1) / kWave, S);
    k_phi_consts<<<g, kWave, 0, stream>>>(P, S, phi, pk, pkr);
    return hipGetLastError();
}

hipError_t launch_windows(const ProbDev &P, int S, const double *phi, int *lo,
                          int *hi, const int *perm, hipStream_t stream,
                          float4 *psec) {
    const size_t n = (size_t)S * P.T;
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (P.sec)
        k_windows<true><<<(unsigned)blocks, 256, 0, stream>>>(P, S, phi, lo, hi,
                                                              perm, psec);
    else
        k_windows<false><<<(unsigned)blocks, 256, 0, stream>>>(P, S, phi, lo, hi,
                                                               perm, nullptr);
    return hipGetLastError();
}

// The window step.  Windowed with a constant width it also finds the
// phases' extremes over the samples (for launch_plan, which follows it).
hipError_t launch_peak_plan(const ProbDev &P, const StepDev &st,
                            const double *phi, hipStream_t stream) {
    if (P.cutoff == 0.0 && !P.sec) return hipSuccess;
    if (P.cutoff > 0.0 && !P.sec && st.cab) {
        const int next = (P.K + kWave - 1) / kWave;
        size_t blocks = ((size_t)st.S * P.T + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        if (blocks == 0) blocks = 1;
        k_windows_ext<<<(unsigned)(next + blocks), kCandThreads, 0, stream>>>(P, st, phi,
                                                                              next);
        return hipGetLastError();
    }
    return launch_windows(P, st.S, phi, P.cutoff > 0.0 ? st.lo : nullptr,
                          st.hi, nullptr, stream, P.sec ? st.psec : nullptr);
}

// Windowed mode with a constant width: the candidate ranges of each (tile,
// phase) over the step's samples, from the phases' extremes that
// launch_peak_plan found (the windowed forward tile then finds its exact
// ranges among them).
hipError_t launch_plan(const ProbDev &P, const StepDev &st, hipStream_t stream) {
    if (P.cutoff > 0.0 && !P.sec && st.cab) {
        dim3 g((P.K + kCandThreads - 1) / kCandThreads, P.ntiles);
        k_cand<<<g, kCandThreads, 0, stream>>>(P, st);
    }
    return hipGetLastError();
}

// Dense: one fused forward + adjoint launch.  Windowed: the forward writes
// the residual, the peak-major adjoint follows when `grad` is set.
template <bool ASYM, bool SEC>
static void launch_fused_t(const ProbDev &P, const StepDev &st, bool grad,
                           float *f_out, hipStream_t stream, const ElboOut *elbo) {
    if (P.cutoff > 0.0) {
        dim3 g(P.ntiles, st.S);
        StepDev sf = st;
        if (!grad) sf.rres = nullptr;
        // records in grid steps on a uniform grid (constant width only)
        if (!SEC && uses_grid_steps(P))
            k_win<ASYM, SEC, !SEC><<<g, kBlock, 0, stream>>>(P, sf, f_out);
        else
            k_win<ASYM, SEC, false><<<g, kBlock, 0, stream>>>(P, sf, f_out);
        if (grad) {
            dim3 ga(P.K, st.S + 1);
            const ElboOut out = elbo ? *elbo : ElboOut{};
            if (P.few) k_adjoint_win<ASYM, SEC, kWave><<<ga, kBlock, 0, stream>>>(P, st, out);
            else k_adjoint_win<ASYM, SEC, kAdjLanes><<<ga, kBlock, 0, stream>>>(P, st, out);
        }
    } else {
        const DenseCut cut = dense_cut(P.N, st.S);
        auto run_cut = [&](auto sg_tag, auto lv_tag, auto cut_tag) {
            constexpr int SG = decltype(sg_tag)::value, LV = decltype(lv_tag)::value;
            constexpr bool CUT = decltype(cut_tag)::value;
            constexpr int nt = kDenseWaves * kWave;
            const int w = cut.wide(P.N);
            const dim3 g(st.nt, (st.S + SG - 1) / SG);
            if (grad) k_dense<true, ASYM, SEC, SG, LV, CUT><<<g, nt, 0, stream>>>(P, st, f_out, w);
            else k_dense<false, ASYM, SEC, SG, LV, CUT><<<g, nt, 0, stream>>>(P, st, f_out, w);
        };
        auto run = [&](auto sg_tag, auto lv_tag) {
            constexpr int SG = decltype(sg_tag)::value, LV = decltype(lv_tag)::value;
            if (direct_peaks<SG, ASYM>(P.K, P.T)) {
                const dim3 g(st.nt, (st.S + SG - 1) / SG);
                const int w = cut.wide(P.N);
                if (grad)
                    k_direct<true, ASYM, SEC, SG, LV>
                        <<<g, kDenseWaves * kWave, 0, stream>>>(P, st, f_out, w);
                else
                    k_direct<false, ASYM, SEC, SG, LV>
                        <<<g, kDenseWaves * kWave, 0, stream>>>(P, st, f_out, w);
            } else if (cut_phases(P.K)) run_cut(sg_tag, lv_tag, std::true_type{});
            else run_cut(sg_tag, lv_tag, std::false_type{});
        };
        const std::integral_constant<int, 1> one;
        const std::integral_constant<int, 2> two;
        const std::integral_constant<int, 4> four;
        if (cut.leaves == 4) run(four, four);
        else if (cut.group == 4) run(four, two);
        else run(one, two);
    }
}

hipError_t launch_fused(const ProbDev &P, const StepDev &st, bool grad,
                        float *f_out, hipStream_t stream, const ElboOut *elbo) {
    if (P.D == 5) {
        if (P.sec) launch_fused_t<true, true>(P, st, grad, f_out, stream, elbo);
        else launch_fused_t<true, false>(P, st, grad, f_out, stream, elbo);
    } else {
        if (P.sec) launch_fused_t<false, true>(P, st, grad, f_out, stream, elbo);
        else launch_fused_t<false, false>(P, st, grad, f_out, stream, elbo);
    }
    return hipGetLastError();
}

hipError_t launch_elbo(const ProbDev &P, const StepDev &st, const ElboOut &out,
                       hipStream_t stream) {
    if (P.cutoff > 0.0) k_elbo<kBlock><<<1, kBlock, 0, stream>>>(P, st, out);
    else k_elbo<1024><<<1, 1024, 0, stream>>>(P, st, out);
    return hipGetLastError();
}

hipError_t launch_grad(const ProbDev &P, const StepDev &st, double scale,
                       const double *scale_dev, double *gloc,
                       double *glogscale, hipStream_t stream,
                       double *gz_out) {
    if (P.cutoff > 0.0)
        k_grad_win<<<(P.K + kWaves - 1) / kWaves, 256, 0, stream>>>(
            P, st, scale, scale_dev, gloc, glogscale, gz_out);
    else
        k_grad<<<P.K, 256, 0, stream>>>(P, st, scale, scale_dev, gloc, glogscale,
                                        gz_out);
    return hipGetLastError();
}

hipError_t launch_adam(int n, double *theta, double *m1, double *m2,
                       const double *g, int t, double lr, double b1, double b2,
                       double eps, hipStream_t stream) {
    k_adam<<<(n + 255) / 256, 256, 0, stream>>>(n, theta, m1, m2, g, t, lr, b1,
                                                 b2, eps);
    return hipGetLastError();
}

}  // namespace xrdvi

namespace xrdvi {

// Log posterior density ln p(Y|phi) + ln p(phi) + ln|J| and its gradient in
// z at the positions z [S][D K] (one per sample): the sampling step with a
// zero mean and unit scale reproduces z exactly, the rest is the ELBO
// step's fused forward, adjoint and chain rule, with per-sample outputs.
hipError_t launch_logpost(const ProbDev &P, const StepDev &st,
                          const double *zeros, const double *z, double *logp,
                          double *gz, hipStream_t stream) {
    hipError_t e = launch_sample(P, st, zeros, zeros, z, 0, 0, stream);
    if (e == hipSuccess) e = launch_peak_plan(P, st, st.phi, stream);
    if (e == hipSuccess) e = launch_plan(P, st, stream);
    const ElboOut el{zeros, nullptr, nullptr, logp};
    if (e == hipSuccess) e = launch_fused(P, st, gz != nullptr, nullptr, stream, &el);
    if (e == hipSuccess && !elbo_in_fused(P, gz != nullptr)) e = launch_elbo(P, st, el, stream);
    if (e == hipSuccess && gz)
        e = launch_grad(P, st, 1.0, nullptr, nullptr, nullptr, stream, gz);
    return e;
}

}  // namespace xrdvi
