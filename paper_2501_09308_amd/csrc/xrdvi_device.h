// Device-side layout and per-tile work of the xrdvi hot path (gfx950).
//
// One step of the method over S Monte-Carlo samples (Sec. 3.2, App. A):
//   sample   z = loc + exp(logscale) eps, phi = T(z), log prior + log|J|
//   windows  per (sample, peak): grid range inside rho +- c w (FP64 bounds)
//   forward  per (2-theta tile, sample): profile f = B + sum_k h_k C_k in
//            FP32, Poisson log-likelihood and residual y/f - 1 in FP64
//   adjoint  recomputes the peak values and accumulates six FP32 sums per
//            (sample, phase) -- the S x K x N basis is never stored; dense in
//            the forward's launch (dense_tile.h), windowed peak by peak
//   grad     FP64 reduction of the tile sums in fixed order and the chain
//            rule to (loc, logscale)
//   elbo     FP64 assembly of the estimate
//
// Peak shape (Appendix A.2, pseudo-Voigt): with q2 = 2 (x - rho) / w,
//   G = (cG / w) 2^(-q2^2),  L = (cL / w) / (1 + q2^2),
//   cG = 2 sqrt(ln2 / pi), cL = 2 / pi
// (unit-area Gaussian and Lorentzian of full width at half maximum w).
//
// Asymmetric peaks (Appendix A.2, asymmetry factor A(x; alpha): alpha on the
// high-angle side of the peak, 1 below it): the full width is w below rho
// and alpha w from rho up, and the peak is scaled by 2 / (1 + alpha) so that
// it keeps unit area; the same formulas hold with q2 = 2 (x - rho) / (A w)
// and the prefactors multiplied by 2 / (1 + alpha).  Each phase then has a
// fifth latent, alpha = exp(z_alpha) with a normal prior.
//
// Angle-dependent width (Appendix A.2 uses sec(x) = 1/cos(x) in the lost
// width formula): with the sec law the full width of peak m of phase k is
// W = w sec(theta), theta = rho / 2, taken as w / |cos(rho pi / 360)|.
// Writing c = |cos theta|, the peak is the same function of
// q2 = 2 c (x - rho) / (A w) with its intensity scaled by c, so the phase
// constants stay per phase and each peak carries (c, I c); the shift's
// gradient gains the term of dW/drho = W tan(theta) pi / 360.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace xrdvi {

constexpr int kWave = 64;
constexpr int kPPL = 2;                   // 2-theta points per lane
constexpr int kTile = kWave * kPPL;       // points per tile (one block)
constexpr int kWaves = 4;                 // waves per block, splitting phases
constexpr int kBlock = kWave * kWaves;
// Points per reference position of a dense problem's positions and grid (the
// windowed: kTile): the widest dense tile, so that its peaks have one offset.
constexpr int kRefDense = 256;
// The Gaussian term of a peak is evaluated only within kGaussReach FWHM of its
// centre: beyond 4.6 w, 2^(-q2^2) < 2^-84 of the peak height, below half an FP32
// unit of the profile (f >= B > 0) for every peak up to 1e18 times the
// background.  A nearer end shows: at 3.5 w (2^-49) a purely Gaussian peak of
// 1e6 counts on a background of 1e-6 is off by 1e-3 just past it, and saves only
// 1 to 5 % (200 x 60 peaks dense, N = 7001, S = 128 687 us for 726; 2000 x 100,
// N = 14001, windows of 8 FWHM 1261 for 1277).
constexpr double kGaussReach = 4.6;

constexpr double kCG = 0.93943727869965133377;   // 2 sqrt(ln 2 / pi)
constexpr double kCL = 0.63661977236758134308;   // 2 / pi
constexpr double kLn2 = 0.69314718055994530942;
constexpr double kLn2Pi = 1.83787706640934548356;  // ln(2 pi)
constexpr double kTwoPi = 6.28318530717958647693;
constexpr double kHalfDegRad = 3.14159265358979323846 / 360.0;  // rad per deg / 2

// A prepared problem in device memory (peaks ordered by position within
// each phase).
struct ProbDev {
    int N, K, T, ntiles;
    int ref;                          // points that share a reference point xref:
                                      // a tile, or 256 (kRefDense) in dense mode
    int D;                            // latent types per phase: 4, or 5 with
                                      // the asymmetry alpha
    int sec;                          // 1: width w sec(rho / 2); 0: width w
    int few;                          // 1: no phase has more than kAdjFew peaks
    double cutoff;
    double lambda, mu_sd, w_shape, w_rate;
    double a_mean, a_sd;              // normal prior on alpha (D = 5)
    // log-density constants: ln lambda, -ln(mu_sd sqrt(2 pi)),
    // shape ln(rate) - lgamma(shape), -ln(a_sd sqrt(2 pi))
    double c_h, c_mu, c_w, c_a;
    const double *x, *y, *bg, *lgy;   // [N]; lgy = ln y!
    double x0, inv_dx;                // x[0] and (N - 1) / (x[N-1] - x[0])
                                      // (0 for N = 1): grid-search guesses
    double dx;                        // (x[N-1] - x[0]) / (N - 1) (0 for N = 1)
    int uniform;                      // 1: every x_i lies within 1e-9 dx of
                                      // x0 + i dx
    int formed_x;                     // 1: the windowed adjoint forms x_i
                                      // instead of loading it (a uniform
                                      // grid; symmetric peaks of constant
                                      // width, whose q2 it then forms in
                                      // FP32, only with windows of at most
                                      // kF32Cutoff FWHM)
    const float *u;                   // [ntiles * kTile] x_i - xref (of ref points)
                                      // (FP32, rounded)
    const float *ul;                  // [ntiles * kTile] its rounding
                                      // error: (x_i - xref) - u_i in FP32
    const int *off;                   // [K + 1]
    const int *phase;                 // [T] phase of each peak
    const double *pos;                // [T]
    const float *inten;               // [T]
    const float *pt;                  // [ceil(N / ref)][T] p_j - xref
    const float *ptl;                 // [ceil(N / ref)][T] its rounding error
    // position index of each phase's sorted peaks: ptab[k][b] is the first
    // peak j of phase k with pos[j] >= tab_x0 + b / tab_inv (b = 0 ..
    // kTabBuckets), a starting guess for searches over positions
    const int *ptab;
    double tab_x0, tab_inv;
    const int2 *near;         // dense mode, constant widths: table of near ranges of
    int near_kinds;           // so many kinds of tiles and margins (dense_tile.h)
    int near_levels;
};

constexpr int kTabBuckets = 128;

// Per-step state of one analysis with S samples.
// Number of adjoint sums per (sample, phase): six, or six per side of the
// peak (below / above rho) for asymmetric peaks.
__host__ __device__ inline int num_sums(int D) { return D == 5 ? 12 : 6; }

struct StepDev {
    int S;
    int nt;           // tiles of the likelihood and adjoint sums: P.ntiles, or in
                      // dense mode those of dense_cut
    int near_levels;  // dense mode: margins looked up (near_shape)
    double *eps;      // [S][D K] noise used
    double *phi;      // [S][D K] constrained samples (h, mu, w, r[, alpha])
    float4 *pk;       // [S][K] (2/w, h(1-r)cG n/w, h r cL n/w, mu) in FP32,
                      // n = 2/(1+alpha) (1 for symmetric peaks)
    float *pkr;       // [S][K] 2/(alpha w): the high-angle side (D = 5)
    double *lpj;      // [S][K] log prior + log|J|
    double *lpb;      // [S][ceil(K/64)] per-wave sums of lpj
    int *lo, *hi;     // [S][T] window plan (sorted peak order)
    float4 *psec;     // [S][T] sec width law, per (sample, peak):
                      // (c, I c, tan(theta) (pi/360) w, 0), c = |cos theta|
    float *rres;      // [S][N] residual y/f - 1 (windowed mode; dense: null)
    double *pw;       // [K][S][num_sums] adjoint sums per (phase, sample)
                      // (windowed mode)
    double *llp;      // [S][nt] per-tile log-likelihood
    float *part;      // [nt][K][S][num_sums] adjoint tile sums
    double *sd;       // [D K] exp(logscale)
    // windowed mode, constant width: the candidate peaks of each (tile,
    // phase) over the step's samples, laid out [..][ntiles][K] so that the
    // forward's threads (one per phase of a tile) read them coalesced:
    int2 *cab;        // [ntiles][K] candidates [ca, cb)
    float4 *cp;       // [ntiles][K] tile-relative positions of the first four
    double4 *cext;    // [K] (min mu, max mu, max w, max w alpha) over samples
};

// Read-only view of data that no kernel of the current launch writes:
// uniform loads through it become scalar loads.
template <typename T>
using cptr = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T *p) {
    return (cptr<T>)p;
}

__device__ __forceinline__ float rcp_f32(float v) {
    return __builtin_amdgcn_rcpf(v);
}
__device__ __forceinline__ float exp2_f32(float v) {
    return __builtin_amdgcn_exp2f(v);
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

__device__ __forceinline__ int wave_max_i32(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, kWave));
    return v;
}

// ---- Philox4x32-10 (Salmon et al., SC'11) + Box-Muller ------------------

__device__ __forceinline__ void philox10(uint32_t c[4], uint32_t k0,
                                         uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t a = c[0], b = c[2];
        const uint32_t hiA = __umulhi(0xD2511F53u, a), loA = 0xD2511F53u * a;
        const uint32_t hiB = __umulhi(0xCD9E8D57u, b), loB = 0xCD9E8D57u * b;
        c[0] = hiB ^ c[1] ^ k0;
        c[1] = loB;
        c[2] = hiA ^ c[3] ^ k1;
        c[3] = loA;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Standard normal number j of sample s at (seed, step): Philox block j/4,
// uniform pair (j & 3) >> 1, cosine branch for even j, sine for odd j.
__device__ inline double philox_normal(uint64_t seed, uint64_t step, int s,
                                       int j) {
#pragma clang fp contract(off)
    uint32_t c[4] = {(uint32_t)(j >> 2), (uint32_t)s, (uint32_t)step,
                     (uint32_t)(step >> 32)};
    philox10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    const int pr = (j & 3) >> 1;
    const double ua = ((double)c[2 * pr] + 0.5) * 2.3283064365386962890625e-10;
    const double ub = ((double)c[2 * pr + 1] + 0.5) * 2.3283064365386962890625e-10;
    const double rad = sqrt(-2.0 * log(ua));
    const double ang = kTwoPi * ub;
    return (j & 1) ? rad * sin(ang) : rad * cos(ang);
}

// ---- transforms and priors (Sec. 2.2, Sec. 3.2, Appendix B.2) ----------

__device__ __forceinline__ double softplus(double a) {
    return a > 0.0 ? a + log1p(exp(-a)) : log1p(exp(a));
}

// FP32 kernel constants of one (sample, phase).
// nrm = 2 / (1 + alpha) for asymmetric peaks, 1 otherwise.  The kernels
// evaluate the Gaussian as 2^(-tt) = 2^(-1 - q2^2) with tt = 1 + q2^2 (the
// Lorentzian's denominator, and the exponent's negation is free), so its
// amplitude here is twice h (1 - r) cG n / w, and the adjoint's Gaussian
// sums are half those of 2^(-q2^2) (phase_grad doubles them).
__device__ __forceinline__ float4 phase_consts(double h, double mu, double w,
                                               double r, double nrm = 1.0) {
    const double iw = 1.0 / w;
    return make_float4((float)(2.0 * iw),
                       (float)(2.0 * h * (1.0 - r) * kCG * iw * nrm),
                       (float)(h * r * kCL * iw * nrm), (float)mu);
}
__device__ __forceinline__ double asym_norm(double alpha) {
    return 2.0 / (1.0 + alpha);
}
__device__ __forceinline__ float asym_iw2(double w, double alpha) {
    return (float)(2.0 / (alpha * w));
}

// ---- window plan ---------------------------------------------------------

// Grid searches.  The grid is ascending and usually close to uniform, so a
// search starts at the index a uniform grid would give and checks the true
// values there (grid_range below); the result is the exact bound for any
// ascending grid.

// Index guess for value v on a grid starting at x0 with inv_dx points per
// unit (clamped to [0, n]; NaN gives 0).
__host__ __device__ inline int grid_guess(double x0, double inv_dx, int n,
                                          double v) {
    const double g = (v - x0) * inv_dx;
    if (!(g > 0.0)) return 0;
    if (!(g < (double)n)) return n;
    return (int)g;
}

// Batched searches.  A search from a good guess costs one round trip to
// memory when the entries around the guess are loaded together: a probe
// loads NP consecutive entries from j0 (several searches issue their probes
// before any result is needed), and the answer is read off the probe when
// it lies inside.  Otherwise the search moves a whole probe towards it (two
// more probes at most) and bisects what remains.  Entries are read clamped
// to [a, b - 1] (entry 0 when the range is empty), so every load stays in
// bounds for any j0.
template <int NP, typename T>
struct Probe {
    int j0;
    T v[NP];
};

template <int NP, typename T>
__host__ __device__ __forceinline__ Probe<NP, T> probe_at(const T *v, int a,
                                                         int b, int j0) {
    Probe<NP, T> p;
    p.j0 = j0;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int j = j0 + i < a ? a : (j0 + i > b - 1 ? b - 1 : j0 + i);
        p.v[i] = v[a < b ? j : 0];
    }
    return p;
}

// The number of leading entries of a probe (loaded by probe_at with the
// same a and b) whose predicate is false, pred false and then true over
// [a, b): entries below a count as false and entries at or past b as true.
// Evaluating every probe this way first leaves one integer per search live
// instead of the probed values.
template <int NP, typename T, typename F>
__host__ __device__ __forceinline__ int probe_count(const Probe<NP, T> &p,
                                                   int a, int b, F pred) {
    int nf = 0;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int j = p.j0 + i;
        nf += (j >= b || (j >= a && pred(p.v[i]))) ? 0 : 1;
    }
    return nf;
}

// First j in [a, b) with pred(v[j]) true, b if none, given the count nf of
// a probe at j0: the answer j0 + nf when it lies inside the probe, otherwise
// the search goes on by whole probes (two more at most), then bisects.
template <int NP, typename T, typename F>
__host__ __device__ inline int probe_settle(const T *v, int a, int b, int j0,
                                            int nf, F pred) {
    if (a >= b) return a;
    int lo = a, hi = b;                     // the answer lies in [lo, hi]
    for (int round = 0;; ++round) {
        if (nf > 0 && nf < NP) return j0 + nf;
        if (nf == 0) hi = j0 < hi ? j0 : hi;               // at or left of j0
        else lo = j0 + NP > lo ? j0 + NP : lo;             // right of the probe
        if (lo >= hi || round == 2) break;
        j0 = nf == 0 ? (hi - NP > lo ? hi - NP : lo) : lo;
        nf = probe_count(probe_at<NP>(v, a, b, j0), a, b, pred);
    }
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (pred(v[mid])) hi = mid; else lo = mid + 1;
    }
    return lo;
}

template <int NP, typename T, typename F>
__host__ __device__ inline int probe_result(const T *v, int a, int b,
                                            const Probe<NP, T> &p, F pred) {
    return probe_settle<NP>(v, a, b, p.j0, probe_count(p, a, b, pred), pred);
}

// Grid range [lo, hi) of the points with va <= x_i <= vb (lo = first i with
// x[i] >= va, hi = first i with x[i] > vb; both written as negated "before"
// tests, so a NaN bound gives 0), each bound from a two-point probe at the
// uniform-grid guess.  grid_probe issues both probes, grid_finish reads the bounds off
// them, so that the probes of several ranges can be in flight together.
struct GridProbe {
    Probe<2, double> a, b;
    double va, vb;
};
__host__ __device__ __forceinline__ GridProbe grid_probe(const double *x, int n,
                                                        double x0, double inv_dx,
                                                        double va, double vb) {
    return GridProbe{probe_at<2>(x, 0, n, grid_guess(x0, inv_dx, n, va)),
                     probe_at<2>(x, 0, n, grid_guess(x0, inv_dx, n, vb)), va, vb};
}
__host__ __device__ inline int2 grid_finish(const double *x, int n,
                                            const GridProbe &g) {
    const double va = g.va, vb = g.vb;
    auto ge = [&](double xi) { return !(xi < va); };
    auto gt = [&](double xi) { return !(xi <= vb); };
    const int na = probe_count(g.a, 0, n, ge), nb = probe_count(g.b, 0, n, gt);
    return make_int2(probe_settle<2>(x, 0, n, g.a.j0, na, ge),
                     probe_settle<2>(x, 0, n, g.b.j0, nb, gt));
}
__host__ __device__ inline int2 grid_range(const double *x, int n, double x0,
                                           double inv_dx, double va,
                                           double vb) {
    return grid_finish(x, n, grid_probe(x, n, x0, inv_dx, va, vb));
}

// The window's bounds a = rho - c W and b = rho + c W (rho + (c W) alpha for
// asymmetric peaks, alpha > 0), rho = p + mu, W the peak's full width; each is
// one rounded FP64 operation (no contraction), as in the model's definition.
__device__ __forceinline__ double2 window_bounds(const ProbDev &P, double p,
                                                 double mu, double W,
                                                 double alpha) {
#pragma clang fp contract(off)
    const double rho = p + mu;
    const double hw = P.cutoff * W;
    return make_double2(rho - hw, rho + (P.D == 5 ? hw * alpha : hw));
}

// Grid points below v on a uniform grid where v itself says so: every x_i is
// within 1e-9 steps of x0 + i dx (ProbDev::uniform), so a v further than
// kGridSure steps from that needs no look at x.  -1: it does (also for NaN and
// infinity).  Saves both bounds' probes, four scattered FP64 loads per window:
// with the indices of windows_elem in 32 bits, 6.4 million windows (2000x100,
// S=32) 59 -> 27 us.
constexpr double kGridSure = 1e-6;
__device__ __forceinline__ int grid_below(const ProbDev &P, double v) {
    const double g = (v - P.x0) * P.inv_dx, fl = floor(g), f = g - fl;
    if (!(f > kGridSure && f < 1.0 - kGridSure)) return -1;
    return g < 0.0 ? 0 : (g > (double)(P.N - 1) ? P.N : (int)fl + 1);
}

// Grid range [lo, hi) of the points within the window's bounds.
__device__ inline int2 window_of(const ProbDev &P, double p, double mu,
                                 double W, double alpha) {
    if (P.cutoff == 0.0) return make_int2(0, P.N);
    const double2 ab = window_bounds(P, p, mu, W, alpha);
    int2 r = make_int2(-1, -1);
    if (P.uniform) r = make_int2(grid_below(P, ab.x), grid_below(P, ab.y));
    if (r.x < 0 || r.y < 0) r = grid_range(P.x, P.N, P.x0, P.inv_dx, ab.x, ab.y);
    if (r.y < r.x) r.y = r.x;
    return r;
}

// ---- per-(sample, tile, phase) peak ranges ---------------------------------
//
// Peaks are ordered by position inside each phase, so for a fixed sample
// the window bounds are monotone in the peak index and both the peaks whose
// window reaches a tile and the peaks whose Gaussian matters there form
// contiguous index ranges.

// First j in [a, b) with p[j] + mu > key (FP64 sum, as the peak centre
// rho is formed everywhere else); monotone because p is sorted.
__device__ inline int first_centre_above(const double *p, int a, int b,
                                         double mu, double key) {
#pragma clang fp contract(off)
    while (a < b) {
        const int mid = (a + b) >> 1;
        if (p[mid] + mu > key) b = mid; else a = mid + 1;
    }
    return a;
}

// Probe start for the first peak of phase k (peaks [a, b)) whose position
// is >= v: one before the bucket's first peak, so that the probe also
// covers an answer one to the left of it.
__device__ __forceinline__ int tab_guess(const ProbDev &P, int k, double v,
                                         int a, int b) {
    const double g = (v - P.tab_x0) * P.tab_inv;
    const int u = !(g > 0.0) ? 0 : (g < (double)kTabBuckets ? (int)g : kTabBuckets);
    const int j = P.ptab[k * (kTabBuckets + 1) + u];
    return (j < a ? a : (j > b ? b : j)) - 1;
}

// ---- candidate ranges (windowed mode, constant width) --------------------
//
// The peaks of a phase whose window reaches a tile at sample s lie among
// those whose window could reach it at any sample of the step: positions p
// with xa - max_s(mu) - c max_s(w alpha) <= p <= xb - min_s(mu) + c max_s(w)
// (widened by a margin far above FP64 rounding).  Found once per step for
// every (tile, phase), so that each (tile, sample) of the windowed forward
// reads them with coalesced loads instead of searching the phase with
// scattered ones.
constexpr int kCandThreads = 256;
// Candidates (or peaks scanned under the sec law) up to which a phase's ranges
// are counted peak by peak; beyond, binary searches of all ends in step.  20
// phases of 300 peaks of 2 deg, windows of 32 deg, N = 3501, S = 32: forward 212
// us counted, 143 searched; 4 of 2000 under the sec law 794 and 292.
constexpr int kCandCount = 16;

// The extremes of each phase over the step's samples: (min mu, max mu,
// max w, max w alpha) to st.cext[k].  Block of kCandThreads threads: 64
// phases (starting at k0) times 4 slices of the samples, combined in LDS.
struct CandExtSmem {
    double v[4][4][kWave];
};
__device__ inline void cand_ext_block(const ProbDev &P, const StepDev &st,
                                      const double *phi, int k0,
                                      CandExtSmem &sm) {
    const int kk = threadIdx.x % kWave, sl = threadIdx.x / kWave;
    const int k = k0 + kk;
    const size_t row = (size_t)P.D * P.K;
    double mn = __builtin_huge_val(), mx = -__builtin_huge_val(), wm = 0.0, wam = 0.0;
    if (k < P.K) {
        for (int s = sl; s < st.S; s += 4) {
            const double mu = phi[s * row + P.K + k], w = phi[s * row + 2 * P.K + k];
            const double al = P.D == 5 ? phi[s * row + 4 * P.K + k] : 1.0;
            mn = fmin(mn, mu);
            mx = fmax(mx, mu);
            wm = fmax(wm, w);
            wam = fmax(wam, w * al);
        }
    }
    sm.v[0][sl][kk] = mn; sm.v[1][sl][kk] = mx; sm.v[2][sl][kk] = wm; sm.v[3][sl][kk] = wam;
    __syncthreads();
    if (sl == 0 && k < P.K) {
#pragma unroll
        for (int o = 1; o < 4; ++o) {
            mn = fmin(mn, sm.v[0][o][kk]);
            mx = fmax(mx, sm.v[1][o][kk]);
            wm = fmax(wm, sm.v[2][o][kk]);
            wam = fmax(wam, sm.v[3][o][kk]);
        }
        st.cext[k] = make_double4(mn, mx, wm, wam);
    }
}

// Candidate range of (tile t, phase k) from the phase's extremes.
__device__ inline void cand_elem(const ProbDev &P, const StepDev &st, int t,
                                 int k) {
#pragma clang fp contract(off)
    const double4 e = st.cext[k];
    const double lo_off = e.y + P.cutoff * e.w;
    const double hi_off = P.cutoff * e.z - e.x;
    const int a = P.off[k], b = P.off[k + 1];
    const int i0 = t * kTile, i1 = min(i0 + kTile, P.N);
    const double xa = P.x[i0], xb = P.x[i1 - 1];
    const double pl = xa - lo_off - (1e-9 + 1e-12 * fabs(xa));
    const double pu = xb + hi_off + (1e-9 + 1e-12 * fabs(xb));
    auto ge = [&](double p) { return !(p < pl); };
    auto gt = [&](double p) { return p > pu; };
    const Probe<4, double> pa = probe_at<4>(P.pos, a, b, tab_guess(P, k, pl, a, b));
    const Probe<4, double> pb = probe_at<4>(P.pos, a, b, tab_guess(P, k, pu, a, b));
    const int na = probe_count(pa, a, b, ge), nb = probe_count(pb, a, b, gt);
    const int ca = probe_settle<4>(P.pos, a, b, pa.j0, na, ge);
    int cb = probe_settle<4>(P.pos, a, b, pb.j0, nb, gt);
    cb = cb < ca ? ca : cb;
    const size_t ci = (size_t)t * P.K + k;
    st.cab[ci] = make_int2(ca, cb);
    const float *pt = P.pt + (size_t)t * P.T;
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = ca + q < cb ? pt[ca + q] : 0.f;
    st.cp[ci] = make_float4(v[0], v[1], v[2], v[3]);
}

// The peaks of phase k that the forward stages for (tile t, sample s): [ja,
// jb), whose windows reach the tile, and [ga, gb) of them, whose Gaussian does
// (constant width).  Counted over the tile's candidates in FP32 tile-relative
// positions with bounds widened far beyond the rounding of their terms: a few
// peaks more than the exact ranges (each record carries its exact window), for a
// quarter of the work of FP64 predicates.  Candidates past the fourth, whose
// positions are not kept beside the range, are read four at a time, and more
// than kCandCount of them searched.
__device__ __forceinline__ int4 cand_ranges(const ProbDev &P, const StepDev &st,
                                            const double *ph, int t, int k,
                                            double xa, double xb, double xref) {
    const size_t ci = (size_t)t * P.K + k;
    const int2 ab = st.cab[ci];
    const float4 cp = st.cp[ci];
    const double mu = ph[P.K + k], w = ph[2 * P.K + k];
    const double al = P.D == 5 ? ph[4 * P.K + k] : 1.0;
    const float a = (float)(xa - xref - mu), b = (float)(xb - xref - mu);
    const float c = (float)(P.cutoff * w), g = (float)(kGaussReach * w), alf = (float)al;
    const float wl = (a - c * alf) - 4e-6f * (1.f + fabsf(a) + c * alf);
    const float wh = (b + c) + 4e-6f * (1.f + fabsf(b) + c);
    const float gl = (a - g * alf) - 4e-6f * (1.f + fabsf(a) + g * alf);
    const float gh = (b + g) + 4e-6f * (1.f + fabsf(b) + g);
    int ja = 0, jb = 0, ga = 0, gb = 0;
    const int n = ab.y - ab.x;
    auto count = [&](int q, float p) {
        const bool in = q < n;
        ja += in && p < wl;
        jb += in && p <= wh;
        ga += in && p < gl;
        gb += in && p <= gh;
    };
    count(0, cp.x); count(1, cp.y); count(2, cp.z); count(3, cp.w);
    const float *pt = P.pt + (size_t)t * P.T + ab.x;
    if (n <= kCandCount) {
        for (int q0 = 4; q0 < n; q0 += 4) {
            float p[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) p[q] = pt[min(q0 + q, n - 1)];
#pragma unroll
            for (int q = 0; q < 4; ++q) count(q0 + q, p[q]);
        }
    } else {
        ja = jb = ga = gb = 0;
        for (int step = 1 << (31 - __clz(n)); step > 0; step >>= 1) {
            auto probe = [&](int j) { return pt[min(j + step, n) - 1]; };
            const float pja = probe(ja), pjb = probe(jb), pga = probe(ga), pgb = probe(gb);
            if (ja + step <= n && pja < wl) ja += step;
            if (jb + step <= n && pjb <= wh) jb += step;
            if (ga + step <= n && pga < gl) ga += step;
            if (gb + step <= n && pgb <= gh) gb += step;
        }
    }
    jb = max(jb, ja);
    ga = min(max(ga, ja), jb);
    gb = min(max(gb, ga), jb);
    return make_int4(ab.x + ja, ab.x + ga, ab.x + gb, ab.x + jb);
}

// The same ranges under the sec law, whose widths grow with the centre: a
// centre below the tile has at most the width at xa, so the first peak follows
// from a search of the positions; from there on the window step's indices tell
// which peaks start past the tile, and the records' c (W = w / c) which
// Gaussians reach it.  No cosine is formed: the phase's first and last records
// say whether the bounds are monotone over its peaks (the whole phase
// otherwise): they move with rho at slopes 1 - R W tau and 1 + R alpha W tau,
// tau = tan(theta) pi / 360, and for centres inside (-180, 180) deg W tau
// increases with rho, so positive slopes at the last and the first centre
// suffice.  cxa: |cos(xa pi / 360)|.
__device__ __forceinline__ int4 sec_ranges(const ProbDev &P, const double *ph, int k,
                                           const int *wlo, const float *psec, int i1,
                                           double xa, double xb, double cxa) {
    const int a = P.off[k], b = P.off[k + 1];
    if (a >= b) return make_int4(a, a, a, a);
    const double mu = ph[P.K + k], w = ph[2 * P.K + k];
    const double al = P.D == 5 ? ph[4 * P.K + k] : 1.0;
    const float4 *ps = reinterpret_cast<const float4 *>(psec);
    const float4 f = ps[a], l = ps[b - 1];
    const double R = fmax(P.cutoff, kGaussReach);
    const double rf = P.pos[a] + mu, rl = P.pos[b - 1] + mu;
    const double up = 1.0 + R * al * f.z / f.x, dn = 1.0 - R * l.z / l.x;
    if (!(rf > -xa && rl < 180.0 && up > 1e-3 && dn > 1e-3)) return make_int4(a, a, b, b);
    const double v = xa - mu - P.cutoff * (w / cxa) * al - 1e-5;
    auto ge = [&](double p) { return !(p < v); };
    const Probe<4, double> pr = probe_at<4>(P.pos, a, b, tab_guess(P, k, v, a, b));
    const int ja = probe_settle<4>(P.pos, a, b, pr.j0, probe_count(pr, a, b, ge), ge);
    int jb = ja, ga = ja, gb = ja;
    const double rw = kGaussReach * w;
    // whether the Gaussian ends below the tile, and begins not above it (both
    // true first, then false)
    auto ends_below = [&](double p, float c) { return p + mu + rw / c * al < xa - 1e-5; };
    auto begins = [&](double p, float c) { return p + mu - rw / c <= xb + 1e-5; };
    bool past = false;
    for (const int stop = min(b, ja + kCandCount); jb < stop && !past;) {
        int lo[4];
        float c[4];
        double p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = min(jb + q, b - 1);
            lo[q] = wlo[j];
            c[q] = ps[j].x;
            p[q] = P.pos[j];
        }
        const int j0 = jb;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            past = past || j0 + q >= b || lo[q] >= i1;
            if (!past) {
                ga += ends_below(p[q], c[q]);
                gb += begins(p[q], c[q]);
                jb = j0 + q + 1;
            }
        }
    }
    if (!past && jb < b) {
        // all of them so far reach the tile: the counts go on from here
        const int j0 = jb, n = b - j0;
        int nj = 0, na = 0, nb = 0;
        for (int step = 1 << (31 - __clz(n)); step > 0; step >>= 1) {
            auto at = [&](int m) { return j0 + min(m + step, n) - 1; };
            const int lj = wlo[at(nj)];
            const double pa = P.pos[at(na)], pb = P.pos[at(nb)];
            const float fa = ps[at(na)].x, fb = ps[at(nb)].x;
            if (nj + step <= n && lj < i1) nj += step;
            if (na + step <= n && ends_below(pa, fa)) na += step;
            if (nb + step <= n && begins(pb, fb)) nb += step;
        }
        jb = j0 + nj;
        if (ga == j0) ga += min(na, nj);
        if (gb == j0) gb += min(nb, nj);
    }
    return make_int4(ja, ga, max(gb, ga), jb);
}

// ---- wave reductions ------------------------------------------------------

template <int CTRL, int ROWS, bool BOUND>
__device__ __forceinline__ float dpp_f32(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v),
                                                      CTRL, ROWS, 0xf, BOUND));
}

// Sum over the 64 lanes with DPP row shifts and row broadcasts (inclusive
// scan inside each row of 16, then across rows); the total ends in lane 63
// and is returned as a wave-uniform value.
__device__ __forceinline__ float wave_total_f32(float v) {
    v += dpp_f32<0x111, 0xf, true>(v);   // row_shr:1
    v += dpp_f32<0x112, 0xf, true>(v);   // row_shr:2
    v += dpp_f32<0x114, 0xf, true>(v);   // row_shr:4
    v += dpp_f32<0x118, 0xf, true>(v);   // row_shr:8
    v += dpp_f32<0x142, 0xa, false>(v);  // row_bcast:15
    v += dpp_f32<0x143, 0xc, false>(v);  // row_bcast:31
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// ---- one phase's peaks over a tile's points, from global memory ------------
//
// The windowed forward's path for phases whose records do not fit the
// staging space (win_tile below).  Per phase the peaks run in segments:
// [ja, ga) and [gb, jb) need only the Lorentzian, [ga, gb) both components.
// For asymmetric peaks [ga, gb) splits further at jr and jl: the tile lies
// above the centres of [ja, jr), straddles those of [jr, jl) and lies below
// those of [jl, jb), so only [jr, jl) picks the width per point.  Each lane is
// masked by the peak's exact window.
struct PeakMask {
    int lo, hi;
    __device__ __forceinline__ float apply(int i, float t) const {
        return (unsigned)(i - lo) < (unsigned)(hi - lo) ? t
                                                        : __builtin_huge_valf();
    }
};

// One peak as a segment loop sees it: tile-relative position (and, for the
// peaks near the tile, the rounding error of that position), intensity,
// its grid window [lo, hi) and, with the sec width law,
// c = |cos theta| and tw = tan(theta) (pi/360) w (the intensity is then
// I c).
struct PeakRec {
    float pt, ptl, I;
    int lo, hi;
    float c, tw;
};

struct SegPeaks {
    cptr<float> pt;       // tile-relative positions
    cptr<float> ptl;      // their rounding errors
    cptr<float> inten;
    cptr<int> wlo, whi;   // windows
    cptr<float> sec;      // per-sample sec-law records, 4 floats each (SEC)
    // scalar loads (unused fields are never loaded)
    template <bool SEC, bool NEAR>
    __device__ __forceinline__ PeakRec rec(int j) const {
        const float l = NEAR ? ptl[j] : 0.f;
        if (SEC)
            return PeakRec{pt[j], l, sec[4 * j + 1], wlo[j], whi[j], sec[4 * j],
                           sec[4 * j + 2]};
        return PeakRec{pt[j], l, inten[j], wlo[j], whi[j], 1.f, 0.f};
    }
};

// Side of a segment: the points lie below the peak centres (or the peaks are
// symmetric), above them, or on both sides (chosen per point).
enum { kBelow = 0, kAbove = 1, kBoth = 2 };

// The lane's points as one phase's segment loops see them (mu: the phase's
// FP32 shift; iw2, iw2r: 2 / (A w) below and above the centre).  Two forms
// of q2 = 2 (x - rho) / (A w) for a peak at tile-relative position pt:
//   far:  q2 = fma(-pt, iw2, uq),                   uq  = (u - mu) iw2,
//   near: q2 = fma(u - pt, iw2, fma(-ptl, iw2, uql)), uql = (ul - mu) iw2.
// The far form carries the rounding of u, pt and uq, an absolute error in
// x - rho of a few 1e-8 times the tile's extent in degrees: harmless where
// q2 is large, but near the centre of a narrow peak, where the Gaussian is
// steep, it would set the profile's error.  The near form subtracts the
// rounded parts first (u - pt is exact or carries only its own relative
// rounding) and adds the small rounding errors ul and ptl separately, so
// that x - rho keeps a relative error of a few units of FP32 rounding.
// Peaks whose Gaussian reaches the tile take the near form (two more VALU
// operations per point), the others the far form.
struct PhasePts {
    float uq[kPPL], uqr[kPPL], uql[kPPL], uqlr[kPPL];
    __device__ __forceinline__ void set(const float (&u)[kPPL],
                                        const float (&ul)[kPPL], float mu,
                                        float iw2, float iw2r, bool asym) {
#pragma unroll
        for (int p = 0; p < kPPL; ++p) {
            const float um = u[p] - mu, ulm = ul[p] - mu;
            uq[p] = um * iw2;
            uql[p] = ulm * iw2;
            uqr[p] = asym ? um * iw2r : uq[p];
            uqlr[p] = asym ? ulm * iw2r : uql[p];
        }
    }
};

// q2 of point p for peak r, and whether the point lies at or above the
// centre (the side of an asymmetric peak).  Sec law: the constant-width q2
// scaled by the peak's c.
struct SegQ {
    float q2;
    bool up;
};
template <int SIDE, bool NEAR, bool SEC>
__device__ __forceinline__ SegQ seg_q(const PeakRec &r, float u,
                                      const PhasePts &pp, int p, float iw2,
                                      float iw2r) {
    float ql = 0.f, qr = 0.f;
    if (NEAR) {
        const float d = u - r.pt;
        if (SIDE != kAbove) ql = fmaf(d, iw2, fmaf(-r.ptl, iw2, pp.uql[p]));
        if (SIDE != kBelow) qr = fmaf(d, iw2r, fmaf(-r.ptl, iw2r, pp.uqlr[p]));
    } else {
        if (SIDE != kAbove) ql = fmaf(-r.pt, iw2, pp.uq[p]);
        if (SIDE != kBelow) qr = fmaf(-r.pt, iw2r, pp.uqr[p]);
    }
    const bool up = SIDE == kAbove || (SIDE == kBoth && ql >= 0.f);
    const float q = SIDE == kBelow ? ql : (SIDE == kAbove ? qr : (up ? qr : ql));
    return SegQ{SEC ? r.c * q : q, up};
}

// Forward terms of the peaks [j0, j1) of one phase: accL += I l, accG += I e
// (GAUSS) with l = 1 / (1 + q2^2), e = 2^(-1 - q2^2) (see phase_consts);
// GAUSS segments take the near form of q2.
template <bool GAUSS, int SIDE, bool SEC, typename PK>
__device__ __forceinline__ void fwd_segment(const PK &pk, int j0, int j1,
                                            const int (&idx)[kPPL],
                                            const float (&u)[kPPL],
                                            const PhasePts &pp,
                                            float iw2, float iw2r,
                                            float (&accL)[kPPL],
                                            float (&accG)[kPPL]) {
#pragma unroll 2
    for (int j = j0; j < j1; ++j) {
        const PeakRec r = pk.template rec<SEC, GAUSS>(j);
        const float I = r.I;
        const PeakMask mk{r.lo, r.hi};
#pragma unroll
        for (int p = 0; p < kPPL; ++p) {
            const float q2 = seg_q<SIDE, GAUSS, SEC>(r, u[p], pp, p, iw2, iw2r).q2;
            const float tt = mk.apply(idx[p], fmaf(q2, q2, 1.0f));
            accL[p] = fmaf(I, rcp_f32(tt), accL[p]);
            if (GAUSS) accG[p] = fmaf(I, exp2_f32(-tt), accG[p]);
        }
    }
}

// Sec law: the shift moves the centre and, through W(rho), the width, so
// the mu sums take per-peak weights (side A: A = 1 below, alpha above):
//   e1 += I e (c q2 + kG (2 ln2 q2^2 - 1)),  kG = A tw / (4 ln2),
//   l1 += I l (c q2 l + kL (1 - 2 l)),       kL = A tw / 4,
// which phase_grad turns into d/dmu exactly as the plain sums (c = 1,
// tw = 0).  With q2^2 = tt - 1 the Gaussian weight is
// c q2 + bG tt + gG, bG = A tw / 2, gG = -A tw (1/2 + 1/(4 ln2)).
struct SecW {
    float bG, gG, kL;
    __device__ __forceinline__ static SecW of(float tws) {
        constexpr float kInv4Ln2 = 0.36067376022224085f;   // 1 / (4 ln 2)
        return SecW{0.5f * tws, -tws * (0.5f + kInv4Ln2), 0.25f * tws};
    }
};

// Point stage of a tile, after the waves' partial signals are in sig:
// f = B + signal in FP64, the tile's Poisson log-likelihood (to st.llp) and
// the residual y/f - 1 (to rres_lds, and to st.rres when it is set).
__device__ __forceinline__ void tile_points(const ProbDev &P, const StepDev &st,
                                            int t, int s, float *f_out,
                                            const float (*sig)[kTile],
                                            float *rres_lds, double *red) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int i0 = t * kTile;
    double ll = 0.0;
    for (int q = threadIdx.x; q < kTile; q += kBlock) {
        const int i = i0 + q;
        float rr = 0.f;
        if (i < P.N) {
            double sg = 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) sg += (double)sig[w][q];
            const double f = P.bg[i] + sg;
            if (f_out) f_out[(size_t)s * P.N + i] = (float)f;
            const double y = P.y[i];
            ll += (y != 0.0 ? y * log(f) : 0.0) - f - P.lgy[i];
            rr = (float)(y / f - 1.0);
            if (st.rres) st.rres[(size_t)s * P.N + i] = rr;
        }
        rres_lds[q] = rr;
    }
    ll = wave_sum(ll);
    if (lane == 0) red[wv] = ll;
    __syncthreads();
    if (threadIdx.x == 0 && st.llp) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) tot += red[w];
        st.llp[(size_t)s * P.ntiles + t] = tot;
    }
}

// ---- windowed forward tile: flat peak records in LDS ------------------------
//
// In windowed mode only one or two peaks of a phase reach a tile, so a loop
// over phases would spend most of its time on per-phase set-up.  The block
// instead stages, 256 phases at a time, one record per peak that reaches the
// tile, holding all that its evaluation needs from its phase: the centre
// relative to the tile, 2 c / (A w) below and above the centre (c = 1 without
// the sec law; A = 1 below, alpha above), the Lorentzian and Gaussian
// amplitudes I h r cL n / w and I h (1 - r) cG n / w (times c with the sec
// law) and the window.  One thread per phase finds its phase's peak ranges
// over the tile and marks a place for each of its peaks in them: those whose
// Gaussian reaches the tile from the front of the list, the others (Lorentzian
// only) from the back, so that each part is evaluated by a loop without a
// per-record branch.  Then all threads write the records, one place each.  The waves then share both parts.  Phases whose records do not
// fit the staging space (they come last in the chunk) are evaluated from
// global memory, phase by phase.
constexpr int kWinChunk = kBlock;   // phases staged at a time (one per thread)
// LDS for the staged peak records of a chunk, the same for the
// single-analysis and the batched forward: which phases take the
// global-memory path, and so the order in which a point's terms are summed,
// depends on it, and a served analysis gives the same bits as its
// one-at-a-time run only if both kernels stage alike.  21 KB hold 896
// symmetric or 672 asymmetric records (seven blocks per CU; the asymmetric
// forward's registers hold it to six).
constexpr int kWinRecBytes = 21 * 1024;

// A staged record.  Its FP32 centre relative to the tile is rounded;
// records whose Gaussian reaches the tile also carry that rounding error cl
// (x - rho is then formed as (u - centre) + (ul - cl), or on a uniform grid
// in grid steps as (u - centre) - cl with u exact, see win_record).
// Symmetric records keep the centre times the scale below (without the
// Gaussian) or cl times that scale (with it), so that q2 takes fused
// multiply-adds (see win_record).  The window is kept relative to the
// tile: its first point and length, both in [0, kTile], packed as
// first | length << 16.  One record is read with one address: 24 bytes
// (symmetric) or 32 (asymmetric: the scale above the centre as well).
template <bool ASYM>
struct alignas(8) WinRecord {
    float c, s, aL, aG;   // centre (or centre times s), 2c/(A w) below, amplitudes
    int wnd;              // window: first | length << 16
    float cl;             // the centre's rounding error (times s if symmetric)
    __device__ __forceinline__ float ahi() const { return s; }
    __device__ __forceinline__ static WinRecord make(float c, float s, float aL, float aG,
                                                     int wnd, float, float cl) {
        return WinRecord{c, s, aL, aG, wnd, cl};
    }
};
template <>
struct alignas(16) WinRecord<true> {
    float c, s, aL, aG;
    int wnd;
    float cl;
    float ah;             // 2c/(alpha w): the scale above the centre
    float pad;
    __device__ __forceinline__ float ahi() const { return ah; }
    __device__ __forceinline__ static WinRecord make(float c, float s, float aL, float aG,
                                                     int wnd, float ah, float cl) {
        return WinRecord{c, s, aL, aG, wnd, cl, ah, 0.f};
    }
};

// The window [lo, hi) of grid indices relative to the tile starting at i0,
// clamped to it, as a record holds it.
__device__ __forceinline__ int win_rel(int lo, int hi, int i0) {
    const int rl = min(max(lo - i0, 0), kTile), rh = min(max(hi - i0, 0), kTile);
    return rl | ((rh - rl) << 16);
}

template <bool ASYM>
struct WinSmem {
    static constexpr int kCap = kWinRecBytes / sizeof(WinRecord<ASYM>);
    struct Sums {
        float sig[kWaves][kTile];   // the waves' partial sums at the points
        float rres[kTile];
    };
    // the last chunk's records are consumed before the sums are written
    union {
        WinRecord<ASYM> rec[kCap];
        Sums e;
    };
    int wmax[kWaves], wmaxn[kWaves], wfit[kWaves], wcnt[kWaves], wcntg[kWaves];
    double red[kWaves];
};

// The forward of one phase over the tile's points from global memory
// (phases whose records did not fit the staging space).
template <bool ASYM, bool SEC>
__device__ void win_phase_global(const SegPeaks &sp, int4 r, int2 r2,
                                 float4 cst, float iw2r,
                                 const float (&u)[kPPL], const float (&ul)[kPPL],
                                 const int (&idx)[kPPL], float (&sig)[kPPL]) {
    const int ja = __builtin_amdgcn_readfirstlane(r.x);
    const int ga = __builtin_amdgcn_readfirstlane(r.y);
    const int gb = __builtin_amdgcn_readfirstlane(r.z);
    const int jb = __builtin_amdgcn_readfirstlane(r.w);
    const float iw2 = cst.x, aG = cst.y, aL = cst.z, mu = cst.w;
    PhasePts pp;
    pp.set(u, ul, mu, iw2, iw2r, ASYM);
    float accL[kPPL], accG[kPPL];
#pragma unroll
    for (int p = 0; p < kPPL; ++p) {
        accL[p] = 0.f;
        accG[p] = 0.f;
    }
    if (ASYM) {
        const int jr = __builtin_amdgcn_readfirstlane(r2.x);
        const int jl = __builtin_amdgcn_readfirstlane(r2.y);
        fwd_segment<false, kAbove, SEC>(sp, ja, ga, idx, u, pp, iw2, iw2r, accL, accG);
        fwd_segment<true, kAbove, SEC>(sp, ga, jr, idx, u, pp, iw2, iw2r, accL, accG);
        fwd_segment<true, kBoth, SEC>(sp, jr, jl, idx, u, pp, iw2, iw2r, accL, accG);
        fwd_segment<true, kBelow, SEC>(sp, jl, gb, idx, u, pp, iw2, iw2r, accL, accG);
        fwd_segment<false, kBelow, SEC>(sp, gb, jb, idx, u, pp, iw2, iw2r, accL, accG);
    } else {
        fwd_segment<false, kBelow, SEC>(sp, ja, ga, idx, u, pp, iw2, iw2r, accL, accG);
        fwd_segment<true, kBelow, SEC>(sp, ga, gb, idx, u, pp, iw2, iw2r, accL, accG);
        fwd_segment<false, kBelow, SEC>(sp, gb, jb, idx, u, pp, iw2, iw2r, accL, accG);
    }
#pragma unroll
    for (int p = 0; p < kPPL; ++p)
        sig[p] = fmaf(aL, accL[p], fmaf(aG, accG[p], sig[p]));
}

// One staged record's terms at the lane's points (lane and lane + 64 of
// the tile).  Only the lanes whose point lies in the window take part: a
// half tile the window misses is skipped by the whole wave.
// UNIF (a uniform grid): u holds the points' exact offsets from the
// tile's reference point in grid steps, and the records hold the centre,
// its rounding error and the scales in grid steps as well, so the points
// carry no rounding error of their own.
template <bool ASYM, bool GAUSS, bool UNIF>
__device__ __forceinline__ void win_record(const WinRecord<ASYM> r,
                                           const float (&u)[kPPL],
                                           const float (&ul)[kPPL], int lane,
                                           float (&sig)[kPPL]) {
    const float ah = r.ahi();
    const int d0 = lane - (r.wnd & 0xffff), len = r.wnd >> 16;
#pragma unroll
    for (int p = 0; p < kPPL; ++p) {
        const bool in = (unsigned)(d0 + p * kWave) < (unsigned)len;
        if (GAUSS) {
            if (in) {
                asm volatile("");   // a branch, as below
                float q2;
                if (ASYM) {
                    const float d = UNIF ? (u[p] - r.c) - r.cl
                                         : (u[p] - r.c) + (ul[p] - r.cl);
                    q2 = d * (d >= 0.f ? ah : r.s);
                } else if (UNIF) {
                    // (u - centre) s - cl s, cl s kept in the record
                    q2 = fmaf(u[p] - r.c, r.s, -r.cl);
                } else {
                    // (u - centre) s + (ul s - cl s), cl s kept in the record
                    q2 = fmaf(u[p] - r.c, r.s, fmaf(ul[p], r.s, -r.cl));
                }
                const float tt = fmaf(q2, q2, 1.0f);
                sig[p] = fmaf(r.aL, rcp_f32(tt), sig[p]);
                sig[p] = fmaf(r.aG, exp2_f32(-tt), sig[p]);
            }
        } else if (in) {
            // (an empty volatile statement keeps a short body a branch, which
            // the wave skips when the half misses the window; the compiler
            // would otherwise evaluate it at both halves and select)
            asm volatile("");
            float q2;
            if (ASYM) {
                const float d = u[p] - r.c;
                q2 = d * (d >= 0.f ? ah : r.s);
            } else {
                // u s - centre s, centre s kept in the record (far peaks)
                q2 = fmaf(u[p], r.s, -r.c);
            }
            sig[p] = fmaf(r.aL, rcp_f32(fmaf(q2, q2, 1.0f)), sig[p]);
        }
    }
}

// Block order of the kernels over (tile, sample) grids.  The hardware deals
// consecutive blocks to the 8 XCDs in turn; block b takes (tile, sample)
// pairs from the (b mod 8)-th contiguous run of the tile-major,
// sample-fastest order, so each XCD's L2 holds the peak data near its own
// run of tiles.
constexpr int kXcds = 8;
__device__ __forceinline__ int2 xcd_tile_sample(int b, int ntiles, int S) {
    const int nb = ntiles * S;
    const int per = nb / kXcds, rem = nb % kXcds;
    const int x = b % kXcds, i = b / kXcds;
    const int q = x * per + min(x, rem) + i;
    return make_int2(q / S, q % S);
}
__device__ __forceinline__ int2 xcd_tile_sample(int ntiles, int S) {
    return xcd_tile_sample(blockIdx.x + blockIdx.y * gridDim.x, ntiles, S);
}

// Block order of the windowed forward when S is a multiple of 8: XCD x
// takes samples [x S/8, (x+1) S/8) of every tile, tile by tile.  Its L2 then
// holds the window arrays of its own samples (each staged record reads its
// window's ends from them, one cache line per phase), which tile-major runs
// over all samples overflow when the phases are many.
__device__ __forceinline__ int2 xcd_sample_group(int S) {
    const int b = blockIdx.x + blockIdx.y * gridDim.x;
    const int G = S / kXcds, i = b / kXcds;
    return make_int2(i / G, (b % kXcds) * G + i % G);
}

// Whether the windowed forward stages its records in grid steps: a uniform
// grid of more than one point.
__host__ __device__ inline bool uses_grid_steps(const ProbDev &P) {
    return P.uniform != 0 && P.N > 1;
}

// UNIF (constant width, uniform grid): the staged records and the points
// are in grid steps relative to the tile's reference point (see win_record).
template <bool ASYM, bool SEC, bool UNIF, typename SM>
__device__ void win_tile(const ProbDev &P, const StepDev &st, int t, int s,
                         float *f_out, SM &sm) {
    static_assert(!(UNIF && SEC), "grid-step records need a constant width");
    constexpr int kCap = SM::kCap;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int i0 = t * kTile;
    const int K = P.K;
    const float4 *pkv = st.pk + (size_t)s * K;
    const float *pkrv = ASYM ? st.pkr + (size_t)s * K : nullptr;
    const float *ptt = P.pt + (size_t)t * P.T;
    const int *wlo = st.lo + (size_t)s * P.T;
    const int *whi = st.hi + (size_t)s * P.T;
    const float *psec = SEC ? reinterpret_cast<const float *>(st.psec + (size_t)s * P.T)
                            : nullptr;
    const double *ph = st.phi + (size_t)s * P.D * K;
    const int iref = min(i0 + kTile / 2, P.N - 1);
    const double xref = P.x[iref];   // the tile's reference
    const int i1 = min(i0 + kTile, P.N);
    const double xa = P.x[i0], xb = P.x[i1 - 1];
    SegPeaks sp;
    sp.pt = as_const(ptt);
    sp.ptl = as_const(P.ptl + (size_t)t * P.T);
    sp.inten = as_const(P.inten);
    sp.wlo = as_const(wlo);
    sp.whi = as_const(whi);
    sp.sec = as_const(psec);

    float u[kPPL], ul[kPPL], ug[kPPL];
    int idx[kPPL];
    float sig[kPPL];
#pragma unroll
    for (int p = 0; p < kPPL; ++p) {
        idx[p] = i0 + p * kWave + lane;
        u[p] = P.u[idx[p]];
        ul[p] = P.ul[idx[p]];
        ug[p] = (float)(idx[p] - iref);   // exact
        sig[p] = 0.f;
    }
    const double cxa = SEC ? fabs(cos(xa * kHalfDegRad)) : 1.0;
    // grid steps per degree (uniform grid)
    const double gpd = P.inv_dx;

    for (int c0 = 0; c0 < K; c0 += kWinChunk) {
        const int nk = min(kWinChunk, K - c0);
        // this thread's phase: the peaks [x, w) whose windows reach the tile
        // and, among them, those [y, z) whose Gaussian does
        int4 rg = make_int4(0, 0, 0, 0);
        if (tid < nk) {
            if constexpr (!SEC) {
                // among the step's candidates (written by the candidate kernel)
                rg = cand_ranges(P, st, ph, t, c0 + tid, xa, xb, xref);
            } else {
                rg = sec_ranges(P, ph, c0 + tid, wlo, psec, i1, xa, xb, cxa);
            }
        }
        const int cnt = rg.w - rg.x, cg = rg.z - rg.y;
        // inclusive prefixes over the block of the record counts and of the
        // Gaussian record counts
        int incl = cnt, inclg = cg;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int v = __shfl_up(incl, o, kWave);
            const int vg = __shfl_up(inclg, o, kWave);
            if (lane >= o) { incl += v; inclg += vg; }
        }
        if (lane == kWave - 1) { sm.wcnt[wv] = incl; sm.wcntg[wv] = inclg; }
        __syncthreads();
        for (int w = 0; w < wv; ++w) { incl += sm.wcnt[w]; inclg += sm.wcntg[w]; }
        const int excl = incl - cnt, exclg = inclg - cg, excln = excl - exclg;
        // records of the phases that fit (a prefix of the chunk: incl grows
        // with the phase index).  Records with a Gaussian fill the list from
        // the front, the others from the back, each in phase and peak order.
        // The phase's thread only marks the slots with (phase, peak); the records
        // are then made by all threads, one slot each: phases have 0 to some
        // six peaks on a tile, so a thread per phase making its own left two
        // thirds of the lanes idle (2000 phases, 110 tiles, S = 32: 195 of the
        // forward's 650 us).
        const bool fits = tid < nk && incl <= kCap;
        if (fits) {
            for (int q = 0; q < cnt; ++q) {
                const int j = rg.x + q;
                const bool gauss = j >= rg.y && j < rg.z;
                const int slot = gauss ? exclg + (j - rg.y)
                                       : kCap - 1 - excln -
                                             (j < rg.y ? j - rg.x : q - cg);
                *reinterpret_cast<int2 *>(&sm.rec[slot]) = make_int2(tid, j);
            }
        }
        // staged record counts and number of fitting phases
        const int ng = wave_max_i32(fits ? inclg : 0);
        const int nn = wave_max_i32(fits ? incl - inclg : 0);
        const int nfit = __builtin_popcountll(__ballot(fits));
        if (lane == 0) { sm.wmax[wv] = ng; sm.wmaxn[wv] = nn; sm.wfit[wv] = nfit; }
        __syncthreads();
        int n_g = 0, n_n = 0, n_fit = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            n_g = max(n_g, sm.wmax[w]);
            n_n = max(n_n, sm.wmaxn[w]);
            n_fit += sm.wfit[w];
        }
        n_g = __builtin_amdgcn_readfirstlane(n_g);
        n_n = __builtin_amdgcn_readfirstlane(n_n);
        n_fit = __builtin_amdgcn_readfirstlane(n_fit);

        // The records.  The tile-relative centre comes from the FP64 position
        // and shift (rounded once, its rounding error kept for the records with
        // the Gaussian), the window from the window step's arrays (a load
        // instead of a search: the forward is bound by VALU issue).
        for (int r = tid; r < n_g + n_n; r += kBlock) {
            const bool gauss = r < n_g;
            const int slot = gauss ? r : kCap - 1 - (r - n_g);
            const int2 mark = *reinterpret_cast<const int2 *>(&sm.rec[slot]);
            const int k = c0 + mark.x, j = mark.y;
            const float4 cst = pkv[k];
            const float iw2 = cst.x, iw2r = ASYM ? pkrv[k] : 0.f;
            const double pj = P.pos[j], mu = ph[K + k];
            const float I = SEC ? psec[4 * j + 1] : P.inten[j];
            const float c = SEC ? psec[4 * j] : 1.f;
            const int2 wnd = make_int2(wlo[j], whi[j]);
            // (in grid steps the scales are 2 dx / w: the degree scales
            // times dx)
            const float iw2u = UNIF ? (float)((double)iw2 * P.dx) : iw2;
            const float iw2ru = UNIF ? (float)((double)iw2r * P.dx) : iw2r;
            float alo = iw2u * c, ahi = alo;
            if (ASYM) {
                // centre at or below the tile's first point: the tile lies
                // above it; at or below its last: it straddles it
                const float ar = iw2ru * c;
                const double rho = pj + mu;
                if (!(rho > xa)) alo = ahi = ar;
                else if (!(rho > xb)) ahi = ar;
            }
            const double cxd = (pj - xref) + mu;
            const double cx = UNIF ? cxd * gpd : cxd;   // grid steps if UNIF
            const float cxf = (float)cx;
            // symmetric peaks keep the centre times the scale (records
            // without the Gaussian) or the rounding error of the centre
            // times the scale (with it), so that q2 takes fused
            // multiply-adds (see win_record)
            const int whi_j = wnd.y < wnd.x ? wnd.x : wnd.y;
            const double cld = cx - (double)cxf;
            const float cl = (float)(ASYM ? cld : cld * (double)alo);
            sm.rec[slot] = WinRecord<ASYM>::make(
                ASYM || gauss ? cxf : (float)(cx * (double)alo), alo, I * cst.z,
                gauss ? I * cst.y : 0.f, win_rel(wnd.x, whi_j, i0), ahi, gauss ? cl : 0.f);
        }
        __syncthreads();

        // the waves share the two lists
        // (two records per pass, unrolled by hand: the volatile statements
        // in the record bodies keep the compiler from unrolling)
        const float (&uu)[kPPL] = UNIF ? ug : u;
        int f = wv;
        for (; f + kWaves < n_g; f += 2 * kWaves) {
            const WinRecord<ASYM> r0 = sm.rec[f], r1 = sm.rec[f + kWaves];
            win_record<ASYM, true, UNIF>(r0, uu, ul, lane, sig);
            win_record<ASYM, true, UNIF>(r1, uu, ul, lane, sig);
        }
        if (f < n_g) win_record<ASYM, true, UNIF>(sm.rec[f], uu, ul, lane, sig);
        for (f = wv; f + kWaves < n_n; f += 2 * kWaves) {
            const WinRecord<ASYM> r0 = sm.rec[kCap - 1 - f], r1 = sm.rec[kCap - 1 - f - kWaves];
            win_record<ASYM, false, UNIF>(r0, uu, ul, lane, sig);
            win_record<ASYM, false, UNIF>(r1, uu, ul, lane, sig);
        }
        if (f < n_n) win_record<ASYM, false, UNIF>(sm.rec[kCap - 1 - f], uu, ul, lane, sig);
        // phases that did not fit (every lane finds the same ranges)
        for (int kl = n_fit + wv; kl < nk; kl += kWaves) {
            const int k = c0 + kl;
            int2 rk2 = make_int2(0, 0);
            int4 rk;
            if constexpr (SEC) rk = sec_ranges(P, ph, k, wlo, psec, i1, xa, xb, cxa);
            else rk = cand_ranges(P, st, ph, t, k, xa, xb, xref);
            if (ASYM) {
                rk2.x = first_centre_above(P.pos, rk.y, rk.z, ph[K + k], xa);
                rk2.y = first_centre_above(P.pos, rk2.x, rk.z, ph[K + k], xb);
            }
            win_phase_global<ASYM, SEC>(sp, rk, rk2, pkv[k], ASYM ? pkrv[k] : 0.f,
                                        u, ul, idx, sig);
        }
        __syncthreads();                       // records consumed
    }

#pragma unroll
    for (int p = 0; p < kPPL; ++p) sm.e.sig[wv][p * kWave + lane] = sig[p];
    __syncthreads();
    tile_points(P, st, t, s, f_out, sm.e.sig, sm.e.rres, sm.red);
}

// ---- peak-major adjoint (windowed mode) -----------------------------------
//
// One block of kWaves waves per (sample s, phase k); the phase's peaks go
// in groups of kAdjPeaks consecutive ones, group g to wave g mod kWaves.  A
// wave takes a group's peaks side by side, kAdjLanes lanes each, over
// consecutive points of their windows (in problems of short peak lists one peak
// on all lanes: kAdjFew); x - rho is formed in FP64 and rounded
// to FP32 (its sign picks the side of an asymmetric peak), or for symmetric
// peaks of constant width on a uniform grid from FP32 offsets each rounded
// once (adjoint_phase).  Six sums (twelve: six per side) accumulate per lane
// over the wave's peaks, are reduced over the wave, then over the waves in
// fixed order.  R = 0 for lanes outside the window (their terms vanish).
// SEC: iw2 and iw2r carry the peak's c, and wl / wh are the mu-sum weights of
// the two sides (see SecW).  The Lorentzian terms and the Gaussian terms are
// two steps, so that a chunk of points where no Gaussian matters skips the
// second.
//
// Bound by instruction issue.  Windows are 20 to 250 points long: with one
// peak's points on all 64 lanes a window of 80 costs 128 and the Gaussian
// (14 of its 16 half-widths squared weigh nothing) is evaluated in every
// chunk; with 16 lanes a peak it costs 80 to 96, the Gaussian in the middle
// half, and one set of per-peak instructions serves four peaks.  Measured,
// 64 lanes -> 16: 50x40, N=3501, S=64 17.0 -> 13.0 us; 2000x100, N=14001,
// S=32 607 -> 510; 300x50 under the sec law, S=32 85 -> 70; 160x50
// asymmetric, S=31 49 -> 37; eight served analyses 206 -> 158 a step.
// (Long windows, or few peaks, keep fewer waves busy: kAdjLong, kAdjFew.)
struct AdjPt {
    float R, q2, tt;
    bool up;
};

// SIDE: where the points of a wave lie about an asymmetric peak's centre, which
// has six sums per side (acc[6 ..]: above); known to lie on one side, they cost
// what a symmetric peak's do.  (Symmetric peaks: kBelow.)

// Adds three of the point's terms to acc[o .. o + 2] (of its side).
template <bool ASYM, int SIDE>
__device__ __forceinline__ void adj_add(float v0, float v1, float v2, bool up, int o,
                                        float (&acc)[ASYM ? 12 : 6]) {
    if constexpr (ASYM && SIDE == kBoth) {
        const float fu = up ? 1.f : 0.f, fd = 1.f - fu;
        acc[o] = fmaf(fd, v0, acc[o]);
        acc[o + 1] = fmaf(fd, v1, acc[o + 1]);
        acc[o + 2] = fmaf(fd, v2, acc[o + 2]);
        acc[o + 6] = fmaf(fu, v0, acc[o + 6]);
        acc[o + 7] = fmaf(fu, v1, acc[o + 7]);
        acc[o + 8] = fmaf(fu, v2, acc[o + 8]);
    } else {
        constexpr int h = ASYM && SIDE == kAbove ? 6 : 0;
        acc[h + o] += v0;
        acc[h + o + 1] += v1;
        acc[h + o + 2] += v2;
    }
}

template <bool ASYM, bool SEC, int SIDE = ASYM ? kBoth : kBelow>
__device__ __forceinline__ void adj_terms_L(float R, float q2, float tt, bool up,
                                            float c, const SecW &wl, const SecW &wh,
                                            float (&acc)[ASYM ? 12 : 6]) {
    const float l = rcp_f32(tt);
    const float Rl = R * l;
    const float Rll = Rl * l;
    float m1L;
    if (SEC) {
        const float kL = up ? wh.kL : wl.kL;
        m1L = fmaf(Rll, fmaf(c, q2, -2.f * kL), Rl * kL);
    } else {
        m1L = Rll * q2;
    }
    adj_add<ASYM, SIDE>(Rl, m1L, Rll, up, 3, acc);
}

template <bool ASYM, bool SEC, int SIDE>
__device__ __forceinline__ AdjPt adj_point_L(float R, float d, float iw2,
                                             float iw2r, float c,
                                             const SecW &wl, const SecW &wh,
                                             float (&acc)[ASYM ? 12 : 6]) {
    const bool up = SIDE == kAbove || (SIDE == kBoth && d >= 0.f);
    const float q2 = d * (up ? iw2r : iw2), tt = fmaf(q2, q2, 1.0f);
    adj_terms_L<ASYM, SEC, SIDE>(R, q2, tt, up, c, wl, wh, acc);
    return AdjPt{R, q2, tt, up};
}

template <bool ASYM, bool SEC, int SIDE = ASYM ? kBoth : kBelow>
__device__ __forceinline__ void adj_point_G(const AdjPt &pt, float c,
                                            const SecW &wl, const SecW &wh,
                                            float (&acc)[ASYM ? 12 : 6]) {
    const float q2 = pt.q2, tt = pt.tt;
    const float Re = pt.R * exp2_f32(-tt);
    const float Req = Re * q2;
    float m1G;
    if (SEC) {
        const float bG = pt.up ? wh.bG : wl.bG;
        const float gG = pt.up ? wh.gG : wl.gG;
        m1G = Re * fmaf(c, q2, fmaf(bG, tt, gG));
    } else {
        m1G = Req;
    }
    adj_add<ASYM, SIDE>(Re, m1G, Req * q2, pt.up, 0, acc);
}

// The Gaussian matters where |x - rho| <= kGaussReach w (the forward's
// rule): 1 + q2^2 <= 1 + (2 kGaussReach)^2.
constexpr float kGaussTT = (float)(1.0 + 4.0 * kGaussReach * kGaussReach);

// Word 3 of a gfx9-family buffer resource (32-bit data format, raw access).
constexpr int kBufferFlags = 0x00020000;

// Peaks a wave handles side by side, and the lanes of each.
constexpr int kAdjPeaks = 4;
constexpr int kAdjLanes = kWave / kAdjPeaks;
// Peaks per phase up to which a problem's adjoint takes one peak at a time on all
// lanes of a wave, so that a short list is spread over the block's waves: 93
// phases of 6 asymmetric peaks, windows of 4000 points, S = 192 772 us a step by
// half the waves, 478 by all; 497 of 3, S = 14 279 and 138; 1000 of 5, windows of
// 133 points, S = 32 134 and 130.
constexpr int kAdjFew = 8;
// Chunks of points whose loads are issued together.
constexpr int kAdjChunks = 4;
// Points in every window of a group from which asymmetric peaks take several
// chunks at once while those lie on one side of the centres: 4 phases of 100
// peaks, windows of 32 deg (N = 3501, S = 32) 155 us a step by single chunks, 135
// so; shorter windows have few such chunks.
constexpr int kAdjLong = 256;

// Windows of at most this many FWHM each side (symmetric peaks of constant
// width on a uniform grid): the adjoint forms q2 = 2 (x - rho) / w in FP32.
// |q2| is at most 2c inside a window and its chunk offsets at most 4c (2c
// from the middle of a window that the grid does not clip), so each of its
// three roundings errs by at most 4c 2^-24: q2 is exact to
// 12c 2^-24, about 6e-6 at c = 8 and 1.1e-5 at this bound (a relative
// gradient error of that order, against a bar of 1e-4).
constexpr double kF32Cutoff = 16.0;

// LN: lanes of a peak, kAdjLanes, or all of the wave in a problem of few peaks
// (ProbDev::few).
template <bool ASYM, bool SEC, int LN>
__device__ inline void adjoint_phase(const ProbDev &P, const StepDev &st,
                                     int s, int k, double (*red)[12]) {
    constexpr int NS = ASYM ? 12 : 6;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int K = P.K;
    const double *ph = st.phi + (size_t)s * P.D * K;
    const double mu = ph[K + k];
    const float iw2 = (float)(2.0 / ph[2 * K + k]);
    const float iw2r = ASYM ? asym_iw2(ph[2 * K + k], ph[4 * K + k]) : iw2;
    // constant width: x - rho is formed already scaled by 2/w in FP64, so
    // that q2 below the centre is one rounding of it (above the centre of an
    // asymmetric peak it is that times 1/alpha); symmetric peaks on a uniform
    // grid take FP32 from there (the chunk loop)
    const double iw2d = 2.0 / ph[2 * K + k];
    const float up_ratio = ASYM ? (float)(1.0 / ph[4 * K + k]) : 1.f;
    // bounded buffer views of the residual and the grid: 32-bit offsets, and
    // reads past the end return 0
    const __amdgpu_buffer_rsrc_t r_rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(st.rres + (size_t)s * P.N), (short)0, P.N * 4, kBufferFlags);
    const __amdgpu_buffer_rsrc_t x_rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)P.x, (short)0, P.N * 8, kBufferFlags);
    const int *wlo = st.lo + (size_t)s * P.T, *whi = st.hi + (size_t)s * P.T;
    const float4 *psec = SEC ? st.psec + (size_t)s * P.T : nullptr;
    const float ka = ASYM ? (float)ph[4 * K + k] : 1.f;
    const bool unif = P.formed_x != 0;
    constexpr int PK = kWave / LN;          // peaks side by side
    const int sub = lane / LN, l = lane % LN;
    const double xl = fma((double)l, P.dx, P.x0);        // uniform grid: x0 + l dx
    const double dxw = LN * P.dx;                 // one chunk of points
    const int a = P.off[k], b = P.off[k + 1];
    float acc[NS];
#pragma unroll
    for (int c = 0; c < NS; ++c) acc[c] = 0.f;
    // the phase's peaks in groups of PK consecutive ones (neighbours
    // in position, with windows of one length), group g to wave g mod 4: only
    // the phase's last group can be short
    for (int j0 = a + PK * wv; j0 < b; j0 += kWaves * PK) {
        const bool ok = j0 + sub < b;
        const int j = ok ? j0 + sub : j0;
        const int lo = wlo[j], hi = whi[j], len = ok ? hi - lo : 0;
        const double rho = P.pos[j] + mu;
        float cq = 1.f, I, tw = 0.f;
        if (SEC) {
            const float4 r = psec[j];
            cq = r.x;
            I = r.y;
            tw = r.z;
        } else {
            I = P.inten[j];
        }
        const SecW wl = SecW::of(tw), wh = SecW::of(tw * ka);
        const float qs = SEC ? iw2 * cq : 1.f, qsr = SEC ? iw2r * cq : up_ratio;
        // points every one of the group's windows has, and the longest window
        int full = __builtin_amdgcn_readlane(len, 0), span = full;
#pragma unroll
        for (int q = 1; q < PK; ++q) {
            const int v = __builtin_amdgcn_readlane(len, q * LN);
            full = min(full, v);
            span = max(span, v);
        }
        // x_i - rho = e + t in FP64.  On a uniform grid x_i is formed, not
        // loaded, so only the residuals are read: e is the lane's offset in
        // one chunk, x0 + (lo + l) dx - rho, and t the chunk's c dx from it;
        // otherwise e = -rho and t = x_i, loaded.  With a constant width e
        // and t carry the factor 2/w (e by a multiply here, c dx by the
        // chunk step, a loaded x_i by a fused multiply-add)
        // the windows' points, one loop per kind of grid
        auto chunks = [&](auto unif_tag) {
            constexpr bool UNIF = decltype(unif_tag)::value;
            // symmetric peaks of constant width on a uniform grid: q2 is
            // formed in FP32 as the chunk's index times the chunk step plus
            // the lane's offset, each rounded once (one fused multiply-add
            // per point instead of an FP64 sum and a conversion; no side of
            // a peak depends on its sign)
            constexpr bool F32 = UNIF && !SEC && !ASYM;
            // the chunk's c dx (scaled by 2/w with a constant width)
            const double step = SEC ? dxw : dxw * iw2d;
            // FP32: chunks counted from the window's middle one, so that the
            // offsets and their roundings are small where the peak is
            const int mid = F32 ? len / (2 * LN) : 0;
            double e = UNIF ? fma((double)(lo + mid * LN), P.dx, xl) - rho : -rho;
            if (!SEC) e *= iw2d;
            const float stepf = (float)step, ef = (float)e;
            double cdx = 0.0;
            float cf = -(float)mid;
            auto load = [&](int c, float &r, double &x) {
                // points past the grid's end read 0
                const int i = lo + l + c;
                r = __uint_as_float(
                    __builtin_amdgcn_raw_buffer_load_b32(r_rs, i * 4, 0, 0));
                if (!UNIF)
                    x = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                                       x_rs, i * 8, 0, 0));
            };
            // sec law: x - rho; constant width: (x - rho) 2/w
            auto offset = [&](double x) {
                return F32 ? fmaf(cf, stepf, ef)
                           : (float)(SEC || UNIF ? e + (UNIF ? cdx : x) : fma(x, iw2d, e));
            };
            auto point = [&](auto side, float R, float d) {
                constexpr int SIDE = decltype(side)::value;
                const AdjPt pt = adj_point_L<ASYM, SEC, SIDE>(R, d, qs, qsr, cq, wl, wh, acc);
                // a wave-uniform branch (a ballot is a scalar value: no
                // lane-to-scalar move); the windows of a group run in step,
                // so their Gaussians matter in the same chunks
                if (__builtin_amdgcn_ballot_w64(pt.tt <= kGaussTT) != 0) {
                    asm volatile("");   // (a branch, not selects)
                    adj_point_G<ASYM, SEC, SIDE>(pt, cq, wl, wh, acc);
                }
                cf += 1.f;
                cdx += step;
            };
            if constexpr (!ASYM) {
                // the chunks from point c on; MASK: some window may end inside
                auto points = [&](auto mask_tag, int c) {
                    constexpr bool MASK = decltype(mask_tag)::value;
                    float rv[kAdjChunks];
                    double xv[kAdjChunks];
#pragma unroll
                    for (int u = 0; u < kAdjChunks; ++u)
                        load(c + u * LN, rv[u], xv[u]);
                    // all loads are issued before the first use, so one
                    // memory latency covers them
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < kAdjChunks; ++u) {
                        if (MASK && c + u * LN >= span) break;
                        float R = rv[u] * I;
                        if (MASK) R = c + u * LN < len - l ? R : 0.f;
                        point(std::integral_constant<int, kBelow>{}, R, offset(xv[u]));
                    }
                };
                int c = 0;
                for (; c + kAdjChunks * LN <= full; c += kAdjChunks * LN)
                    points(std::false_type{}, c);
                for (; c < span; c += kAdjChunks * LN) points(std::true_type{}, c);
            } else {
                // ascending points: the chunks wholly below the four centres,
                // those with points on both sides, those wholly above; the loads
                // two chunks ahead (a lane past its window only adds 0)
                int c = 0;
                float r0, r1, r2;
                double x0 = 0.0, x1 = 0.0, x2 = 0.0;
                auto ahead = [&]() {
                    load(c, r0, x0);
                    load(c + LN, r1, x1);
                };
                auto run = [&](auto side) {
                    constexpr int SIDE = decltype(side)::value;
                    for (; c < span; c += LN) {
                        const float d = offset(x0);
                        const uint64_t above = __builtin_amdgcn_ballot_w64(d >= 0.f);
                        if (SIDE == kBelow && above != 0) break;
                        if (SIDE == kBoth && above == ~0ull) break;
                        load(c + 2 * LN, r2, x2);
                        point(side, c < len - l ? r0 * I : 0.f, d);
                        r0 = r1;
                        r1 = r2;
                        x0 = x1;
                        x1 = x2;
                    }
                };
                // long windows: kAdjChunks chunks at once while all windows have
                // them, on one side of every centre, their Gaussians without a
                // branch between them where they matter in each (one chunk at a
                // time waits on itself where few waves run: 4 phases of 100 peaks
                // of 2 deg, windows of 32 deg, N = 3501, S = 32 155 us, now 131)
                const bool lng = full >= kAdjLong;
                auto runs = [&](auto side) {
                    constexpr int SIDE = decltype(side)::value;
                    for (; c + kAdjChunks * LN <= full; c += kAdjChunks * LN) {
                        float rv[kAdjChunks], dv[kAdjChunks];
                        double xv[kAdjChunks];
#pragma unroll
                        for (int u = 0; u < kAdjChunks; ++u)
                            load(c + u * LN, rv[u], xv[u]);
                        __builtin_amdgcn_sched_barrier(0);
                        const double cdx0 = cdx;
#pragma unroll
                        for (int u = 0; u < kAdjChunks; ++u) {
                            dv[u] = offset(xv[u]);
                            cdx += step;
                        }
                        if (SIDE == kBelow &&
                            __builtin_amdgcn_ballot_w64(dv[kAdjChunks - 1] >= 0.f) != 0) {
                            cdx = cdx0;
                            break;
                        }
                        AdjPt pt[kAdjChunks];
                        uint64_t g[kAdjChunks];
                        bool every = true;
#pragma unroll
                        for (int u = 0; u < kAdjChunks; ++u) {
                            pt[u] = adj_point_L<ASYM, SEC, SIDE>(rv[u] * I, dv[u], qs, qsr, cq,
                                                                 wl, wh, acc);
                            g[u] = __builtin_amdgcn_ballot_w64(pt[u].tt <= kGaussTT);
                            every = every && g[u] != 0;
                        }
                        if (every) {
                            asm volatile("");
#pragma unroll
                            for (int u = 0; u < kAdjChunks; ++u)
                                adj_point_G<ASYM, SEC, SIDE>(pt[u], cq, wl, wh, acc);
                        } else {
#pragma unroll
                            for (int u = 0; u < kAdjChunks; ++u)
                                if (g[u] != 0) {
                                    asm volatile("");
                                    adj_point_G<ASYM, SEC, SIDE>(pt[u], cq, wl, wh, acc);
                                }
                        }
                    }
                };
                if (lng) runs(std::integral_constant<int, kBelow>{});
                ahead();
                run(std::integral_constant<int, kBelow>{});
                run(std::integral_constant<int, kBoth>{});
                if (lng) {
                    runs(std::integral_constant<int, kAbove>{});
                    ahead();
                }
                run(std::integral_constant<int, kAbove>{});
            }
        };
        if (unif)
            chunks(std::true_type{});
        else
            chunks(std::false_type{});
    }
#pragma unroll
    for (int c = 0; c < NS; ++c) acc[c] = wave_total_f32(acc[c]);
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < NS; ++c) red[wv][c] = acc[c];
    }
    __syncthreads();
    if (threadIdx.x < NS) {
        double v = 0.0;
        for (int w = 0; w < kWaves; ++w) v += red[w][threadIdx.x];
        st.pw[((size_t)k * st.S + s) * NS + threadIdx.x] = v;
    }
}

}  // namespace xrdvi
