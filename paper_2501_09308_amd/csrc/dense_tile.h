// Dense mode (c = 0): one (2-theta tile, group of samples) of the fused
// profile + likelihood + adjoint, with the far Lorentzian tails on nodes.
//
// Every peak reaches every point, but a peak whose centre lies at least two
// half-widths of an interval from its middle, and whose Gaussian does not
// reach it, is a smooth function there: the interpolant through kNodes
// Chebyshev nodes of the interval reproduces 1 / (1 + q2^2) to 1.4e-8 of its
// value at the nearest such centre, and the adjoint's l^2 q2 and l^2 to 1e-7
// and 4.3e-7, errors falling by 3.7 per node and faster for farther peaks.
// Two levels of intervals are used: the tile (64 LV points) and its LV leaves
// of 64 points.  Peaks far from the tile (most of them) are evaluated at the
// tile's 16 nodes, peaks far from a leaf only at that leaf's 16 nodes, the
// others at the leaf's points (a peak several times as wide as a leaf is smooth
// enough there to be taken at its nodes wherever it lies: kWide):
//   forward  node sums of all phases, carried from the tile's nodes to the
//            leaves' and from those to the points once per (tile, sample);
//   adjoint  sum_i R_i F(x_i) = sum_n R_n F(v_n) with R_n = sum_i R_i l_n(x_i)
//            (the transpose), so the residual is carried to the nodes once.
//            Every sum is formed of its own terms, the shift's too: the slope
//            of the interpolant of sum I l, whose weights reach 77, in its place
//            had an error of 3.6e-6 where all centres lie well outside the grid
//            (directly 1e-7).
//
// Lanes: a wave holds SG samples (4 or 1).  With SG = 4 the 16 lanes of a
// sample are its nodes and share its points, the peaks are wave-uniform
// (scalar loads) and the adjoint's sums reduce over 16 lanes for four samples
// at once.  SG = 1 is for grids too small to fill the GPU that way: a
// sample's 64 lanes take four far peaks at the tile's 16 nodes together, and
// a leaf's points in one go (so leaves need no nodes).  NW waves split the
// phases, each phase's peaks too where there are few (CUT); very few peaks are
// taken at every point without nodes (dense_direct).
//
// What it measured (one MI355X, step of ELBO, adjoint and gradient, against
// evaluating every peak at every point): 50 phases x 40 peaks, 3501 points,
// S = 64: 208 -> 80 us; 200 x 60, 7001, S = 128: 3611 -> 692 us; asymmetric
// 50 x 50, 2501, S = 32: 160 -> 78 us; profile of 77 x 50, 5003, S = 24: 95 -> 30
// us.  Bound by VALU issue on the large ones (about 80 % of the kernel's cycles;
// the last round of blocks and the stages between the phase loops, some 17 000
// cycles per block, take the rest).
#pragma once

#include "xrdvi_device.h"

namespace xrdvi {

constexpr int kNodes = 16;
constexpr double kFarRadius = 2.0;     // in half-widths of the tile
// Width in half-widths of a leaf from which a peak is taken at its nodes also
// near its centre: poles (at half the width beside the centre) and growth off
// the axis are then those of a peak kFarRadius away.  With every peak near
// taken at the points, peaks of 3 deg (50 x 40, N = 3501, S = 64) took 381 us
// and asymmetric ones (50 x 50, N = 2501, S = 32) 408.
constexpr double kWide = 3.5;
constexpr int kLeaf = kWave;           // points of a leaf
constexpr int kDenseWaves = 16;        // waves per block
constexpr int kPlanPhases = 256;       // phases whose near ranges are held in LDS
constexpr int kNodeStride = kNodes + 1;    // (no LDS bank conflicts)

// Half-width (deg) given to the nodes of a one-point tile.
constexpr double kPointHalf = 0.05;

// The nodes cos(theta_n), theta_n = (2 n + 1) pi / 32, and the numerators
// (-1)^n sin(theta_n) / 16 of their interpolation weights
//   l_n(t) = T16(t) (-1)^n sin(theta_n) / (16 (t - cos theta_n)).
__constant__ const double kNodeCos[kNodes] = {
    0.99518472667219693, 0.95694033573220882,
    0.88192126434835505, 0.77301045336273699,
    0.63439328416364549, 0.47139673682599781,
    0.29028467725446233, 0.09801714032956077,
    -0.098017140329560645, -0.29028467725446216,
    -0.4713967368259977, -0.63439328416364538,
    -0.77301045336273699, -0.88192126434835494,
    -0.95694033573220882, -0.99518472667219682,
};
__constant__ const double kNodeNum[kNodes] = {
    0.0061260712705975377, -0.018142792328403896,
    0.029462296051624853, -0.039649580260227843,
    0.048313153335171062, -0.055120079021772184,
    0.059808770983263058, -0.062199045417012301,
    0.062199045417012308, -0.059808770983263058,
    0.055120079021772191, -0.048313153335171069,
    0.039649580260227843, -0.029462296051624867,
    0.018142792328403899, -0.0061260712705975516,
};
// How a dense analysis is cut into blocks: leaves per tile and samples per
// block (a function of the analysis alone, so that it gives the same bits
// alone and served).
struct DenseCut {
    int leaves, group;
    int narrow = 0;     // four leaves: trailing spans of four cut in twos
    // Tiles of `leaves` leaves; those that follow have two.
    __host__ __device__ int wide(int N) const {
        return (N + leaves * kLeaf - 1) / (leaves * kLeaf) - narrow;
    }
    __host__ __device__ int tiles(int N) const {
        const int w = wide(N);
        return narrow > 0 ? w + (N - w * leaves * kLeaf + 2 * kLeaf - 1) / (2 * kLeaf) : w;
    }
    __host__ __device__ int groups(int S) const { return (S + group - 1) / group; }
    __host__ __device__ long long blocks(int N, int S) const {
        return (long long)tiles(N) * groups(S);
    }
};
__host__ __device__ inline DenseCut dense_cut(int N, int S) {
    // One block of 16 waves runs per CU.  Two leaves while that is one round
    // of the 256 CUs, four beyond: 50 phases of 40 peaks, N = 3501, at 168 to 252
    // blocks of two take 52 us and their 112 to 126 blocks of four 75, at 280 (S =
    // 37) 77.5 and 75.0, at 448 (S = 64) 81 and 76; 200 of 60, N = 7001, at 275
    // 218 and 198.
    if (DenseCut{2, 4}.blocks(N, S) > 256) {
        DenseCut cut{4, 4};
        // A last round that leaves half the CUs idle is shorter with its spans
        // cut in two (a block of two leaves takes some 0.6 of one of four; cut
        // in two everywhere they would cost the other rounds 1.2): 7001
        // points, S = 128, 896 blocks 668 us, 768 wide ones and 248 of two
        // leaves 622.
        const long long over = cut.blocks(N, S) > 256 ? cut.blocks(N, S) % 256 : 0;
        const long long ng = cut.groups(S), x = (over + ng - 1) / ng;
        if (x < cut.wide(N) && 2 * x * ng <= 256) cut.narrow = (int)x;
        return cut;
    }
    // One sample per block (a wave's lanes then take the points, not the nodes:
    // about twice the work on four times the blocks) while one of them runs on each
    // CU, or a little more (two share a CU): 50 x 40, N = 3501, S = 8 (224 blocks)
    // 38.9 us, with four samples 52.3; asymmetric 55 x 57, N = 2566, S = 14 (294), 57
    // steps wide, 102 and 176; S = 16 (448) 45.7 and 52.1, but served with others
    // (their blocks fill the CUs anyway) an analysis costs twice as much: eight, one
    // of them of 448 blocks, 18.0 ms and 21.9.  Short grids, where most peaks are near
    // and few blocks of four samples leave CUs idle, take two on a CU: 35 x 28, N =
    // 200, S = 256 (512 blocks) 88 us and 110, N = 1500, S = 40 (480) 42.9 and 48.1,
    // with peaks of 2 deg 70 and 112; in two rounds N = 300, S = 200 (600) 110 and 97.
    constexpr int kShortGrid = 1536;
    if (DenseCut{2, 1}.blocks(N, S) > (N <= kShortGrid ? 512 : 384)) return DenseCut{2, 4};
    return DenseCut{2, 1};
}

template <int NW, int SG, int LV, bool ASYM, bool SEC>
struct DenseSmem {
    // LDS for the far sums kept for the adjoint (those of the first phases;
    // the others' are formed again): with four samples what one block per CU
    // leaves, 52 phases in tiles of four leaves and 122 in those of two (half
    // as many of asymmetric peaks); with one, 52, and two blocks fit a CU
    static constexpr int kFarFloats = (SG == 4 && LV == 2 ? 92 : 39) * 1024 / 4;
    static constexpr int kPts = LV * kLeaf;
    static constexpr bool kMid = SG == 4;   // peaks are taken at the leaves' nodes
    static constexpr int kFarSums = 3 * (ASYM ? 2 : 1);     // per lane and phase
    static constexpr int kFarCap = kFarFloats / (kFarSums * kWave);
    static_assert(kFarCap >= NW, "a share of a phase has a place");
    static constexpr int kLow = LV * kNodes;     // the leaves' nodes
    float lm[kPts * kNodeStride];         // weights of the leaves' nodes at the points
    float em[kLow * kNodeStride];         // of the tile's at the leaves'
    float us[kPts], ul[kPts];             // points relative to xref, rounding errors
    float sig[NW][SG][kPts];              // the waves' sums at the points
    float nod[NW][kWave + 1];             // ... at the tile's nodes
    float ndl[kMid ? NW : 1][LV][kWave];  // ... at the leaves' nodes
    double pn[SG][kNodes];                // node sums of all waves
    double low[SG][kLow];                 // ... brought to the leaves' nodes; then the
                                          // residual at them
    double rn[SG][kNodes];                // residual at the tile's nodes
    float rres[SG][kPts];                 // residual y/f - 1
    double red[SG * LV];
    int2 nr[kPlanPhases];                 // near peaks [x, y) of each phase
    float far[kFarCap][kFarSums][kWave];
};

// Table of a dense problem of constant widths, made once (launch_prepare), by
// kind of tile (0: two leaves, 1: four):
//   [kinds][levels][tiles][K]  by margin: the peaks of a phase with
//                             |p - middle| < (kFarRadius + margin) half-widths
// An analysis in a server keeps what its cut and S use, a problem of its own
// all.  (The nodes and their weights are formed by each block: a table of
// them takes 96 bytes a point.)
constexpr int kNearLevels = 4;
__host__ __device__ inline double near_margin(int level) {
    return level == 0 ? 0.0625 : level == 1 ? 0.125 : level == 2 ? 0.25 : 0.75;
}
__host__ __device__ inline size_t near_tiles(int N, int kind) {
    const size_t pts = (kind ? 4 : 2) * kLeaf;
    return (N + pts - 1) / pts;
}
// Entries before the rows of (kind, level) in a table of so many levels.
__host__ __device__ inline size_t near_offset(int N, int K, int levels, int kind, int level) {
    return ((kind ? levels * near_tiles(N, 0) : 0) + level * near_tiles(N, kind)) * K;
}
// Kinds of tiles that the cut uses and margins that its steps look up (beyond
// them they search): the table then takes at most 16 S bytes per 128 points and
// phase, no more memory than a plan of each sample's ranges took.  A function
// of N and S alone, as the cut.
struct NearShape {
    int kinds, levels;
    size_t bytes(int N, int K) const {
        return sizeof(int2) * near_offset(N, K, levels, kinds - 1, levels);
    }
};
__host__ __device__ inline NearShape near_shape(int N, int S) {
    const int kinds = dense_cut(N, S).leaves == 4 ? 2 : 1;
    return NearShape{kinds, S > 2 ? kNearLevels : kinds == 2 ? S : 2 * S};
}

// Middle and half-width of the run of points [a, b).
__device__ __forceinline__ double2 mid_half(const ProbDev &P, int a, int b) {
    const cptr<double> x = as_const(P.x);
    const double xa = x[a], xb = x[b - 1];
    return make_double2(0.5 * (xa + xb), b - a > 1 ? 0.5 * (xb - xa) : kPointHalf);
}

// ... of a leaf.  One of a single point has all its nodes there: the tile's
// interpolant, which grows like T16 past the tile's ends, is then taken at the
// point itself (with nodes kPointHalf about it, the far sum at the last of 65
// points in steps of 0.005 deg was off by 3e-5, in steps of 0.001 deg by more
// than itself).
__device__ __forceinline__ double2 leaf_mid_half(const ProbDev &P, int a) {
    const cptr<double> x = as_const(P.x);
    const int b = min(a + kLeaf, P.N);
    const double xa = x[a], xb = x[b - 1];
    return make_double2(0.5 * (xa + xb), 0.5 * (xb - xa));
}

// 1 / d to a rounding or two (d normal), 0 for 0.
__device__ __forceinline__ double inverse(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    return d == 0.0 ? 0.0 : r;
}
__device__ __forceinline__ double cheb16(double t) {
#pragma unroll
    for (int r = 0; r < 4; ++r) t = 2.0 * t * t - 1.0;
    return t;
}
// l_m(t) at t in [-1, 1] (node c, numerator num).
__device__ __forceinline__ float node_weight(double t, double c, double num) {
    const double d = t - c;
    return fabs(d) < 1e-10 ? 1.f : (float)(cheb16(t) * num * inverse(d));
}

// One entry of the near table: tile t of `leaves` leaves, phase k.
__device__ inline int2 dense_near_entry(const ProbDev &P, int leaves, int level, int t, int k) {
    const int ta = t * leaves * kLeaf;
    const double2 h = mid_half(P, ta, min(ta + leaves * kLeaf, P.N));
    const double r = (kFarRadius + near_margin(level)) * h.y;
    int a = P.off[k], b = P.off[k + 1];
    const int end = b;
    for (int lo = a, hi = b; lo < hi;) {
        const int mid = (lo + hi) >> 1;
        if (P.pos[mid] > h.x - r) hi = mid; else lo = mid + 1;
        a = lo;
    }
    for (int lo = a, hi = end; lo < hi;) {
        const int mid = (lo + hi) >> 1;
        if (P.pos[mid] >= h.x + r) hi = mid; else lo = mid + 1;
        b = lo;
    }
    return make_int2(a, b < a ? a : b);
}

// Sum over the LPS consecutive lanes of one sample (16: a DPP row, 32: two
// rows, 64: the wave), valid in the last 16 of them.
template <int LPS>
__device__ __forceinline__ float lanes_total(float v) {
    static_assert(LPS == 16 || LPS == 32 || LPS == 64, "DPP rows");
    v += dpp_f32<0x128, 0xf, true>(v);   // row_ror:8
    v += dpp_f32<0x124, 0xf, true>(v);
    v += dpp_f32<0x122, 0xf, true>(v);
    v += dpp_f32<0x121, 0xf, true>(v);
    if (LPS >= 32) v += dpp_f32<0x142, 0xa, false>(v);   // row_bcast:15
    if (LPS == 64) v += dpp_f32<0x143, 0xc, false>(v);   // row_bcast:31
    return v;
}

// The near peaks [na, nb) of phase k for samples [s0, s0 + ns): those with a
// centre within kFarRadius half-widths of the tile's middle or a Gaussian
// that reaches the tile, at any of the samples (a superset is harmless:
// near peaks are evaluated at every point).
template <bool SEC>
__device__ inline int2 dense_near(const ProbDev &P, const StepDev &st, int t, int leaves,
                                  int k, int s0, int ns, double2 mh) {
    const int a = P.off[k], b = P.off[k + 1];
    if (a >= b) return make_int2(a, a);
    const double xm = mh.x, ha = mh.y, ra = kFarRadius * ha, xa = xm - ha, xb = xm + ha;
    const int K = P.K;
    double lo = __builtin_huge_val(), hi = -__builtin_huge_val();
    bool whole = false;
    // sec law: a centre below xa has at most the width at xa
    const double cxa = SEC ? fabs(cos(xa * kHalfDegRad)) : 1.0;
    for (int g = 0; g < ns; ++g) {
        const double *ph = st.phi + (size_t)(s0 + g) * P.D * K;
        const double mu = ph[K + k], w = ph[2 * K + k];
        const double al = P.D == 5 ? ph[4 * K + k] : 1.0;
        if (SEC) {
            // the reach of a Gaussian is monotone over the phase's peaks (see
            // sec_ranges), from the records of its first and last peak
            const float4 *ps = st.psec + (size_t)(s0 + g) * P.T;
            const float4 f = ps[a], l = ps[b - 1];
            const double rf = P.pos[a] + mu, rl = P.pos[b - 1] + mu;
            const double up = 1.0 + kGaussReach * al * f.z / f.x;
            const double dn = 1.0 - kGaussReach * l.z / l.x;
            whole |= !(rf > -xa && rl < 180.0 && up > 1e-3 && dn > 1e-3);
        }
        const double W = SEC ? w / cxa : w;
        lo = fmin(lo, fmin(xm - ra, xa - kGaussReach * W * al) - mu);
        hi = fmax(hi, fmax(xm + ra, SEC ? xb : xb + kGaussReach * w) - mu);
    }
    if (whole) return make_int2(a, b);
    if (!SEC) {
        // the table's first margin that covers the bounds (one load instead of
        // two searches)
        const double need = fmax(xm - lo, hi - xm) / ha - kFarRadius;
#pragma unroll
        for (int level = 0; level < kNearLevels; ++level)
            if (level < st.near_levels && need < near_margin(level))
                return P.near[near_offset(P.N, K, P.near_levels, leaves == 4, level) +
                              (size_t)t * K + k];
    }
    auto ge = [&](double p) { return p >= lo; };
    auto gt = [&](double p) { return p > hi; };
    const Probe<4, double> pa = probe_at<4>(P.pos, a, b, tab_guess(P, k, lo, a, b));
    const Probe<4, double> pb = probe_at<4>(P.pos, a, b, tab_guess(P, k, hi, a, b));
    const int ca = probe_count(pa, a, b, ge), cb = probe_count(pb, a, b, gt);
    const int na = probe_settle<4>(P.pos, a, b, pa.j0, ca, ge);
    int nb = probe_settle<4>(P.pos, a, b, pb.j0, cb, gt);
    if (SEC) {
        // centres above the tile: on while a Gaussian reaches it
        for (int g = 0; g < ns; ++g) {
            const double *ph = st.phi + (size_t)(s0 + g) * P.D * K;
            const double mu = ph[K + k], w = ph[2 * K + k];
            const float4 *ps = st.psec + (size_t)(s0 + g) * P.T;
            while (nb < b && P.pos[nb] + mu - kGaussReach * w / ps[nb].x <= xb) ++nb;
        }
    }
    return make_int2(na, nb < na ? na : nb);
}

// Weights of the shift's sums under the sec law (side A: A = 1 below the
// centre, alpha above): the shift moves the centre and, through W(rho), the
// width,
//   e1 += I e (c q2 + kG (2 ln2 q2^2 - 1)),  kG = A tw / (4 ln2),
//   l1 += I l (c q2 l + kL (1 - 2 l)),       kL = A tw / 4,
// which phase_grad turns into d/dmu exactly as the plain sums (c = 1,
// tw = 0).  With q2^2 = tt - 1 the Gaussian weight is
// c q2 + bG tt + gG, bG = A tw / 2, gG = -A tw (1/2 + 1/(4 ln2)): SecW.

// Far sums of one phase side at the lane's node: f0 = sum I l, f2 = sum I l^2
// and f1 = sum I l^2 q2, under the sec law (whose shift weights differ by peak)
// sum I (l^2 (c q2 - 2 kL) + l kL) (f1 and f2 with GRAD).
struct FarSums {
    float f0, f1, f2;
};

template <int SLOTS, bool GRAD, bool SEC>
__device__ __forceinline__ FarSums far_sums(cptr<float> pt, cptr<float> inten,
                                            const float4 *ps, int j0, int j1,
                                            int slot, float uq, float iw2,
                                            float ka) {
    FarSums f{0.f, 0.f, 0.f};
    auto add = [&](float p, float I, float c, float tw) {
        float q2 = fmaf(-p, iw2, uq);
        if (SEC) q2 *= c;
        const float l = rcp_f32(fmaf(q2, q2, 1.0f));
        if (GRAD) {
            const float Il = I * l, Ill = Il * l;
            f.f0 += Il;
            f.f2 += Ill;
            if (SEC) {
                const float kL = 0.25f * tw * ka;
                f.f1 = fmaf(Ill, fmaf(c, q2, -2.f * kL), f.f1);
                f.f1 = fmaf(Il, kL, f.f1);
            } else {
                f.f1 = fmaf(Ill, q2, f.f1);
            }
        } else {
            f.f0 = fmaf(I, l, f.f0);
        }
    };
    if (SLOTS == 1) {
#pragma unroll 4
        for (int j = j0; j < j1; ++j) {
            if (SEC) {
                const float4 r = ps[j];
                add(pt[j], r.y, r.x, r.z);
            } else {
                add(pt[j], inten[j], 1.f, 0.f);
            }
        }
    } else {
#pragma unroll 2
        for (int jj = j0; jj < j1; jj += SLOTS) {
            const bool ok = jj + slot < j1;
            const int j = ok ? jj + slot : j0;
            if (SEC) {
                const float4 r = ps[j];
                add(pt[j], ok ? r.y : 0.f, r.x, ok ? r.z : 0.f);
            } else {
                add(pt[j], ok ? inten[j] : 0.f, 1.f, 0.f);
            }
        }
    }
    return f;
}

// A near peak at one sample: its tile-relative centre as a rounded value ch
// and the rest cl (so that x - rho keeps a relative error of a few units of
// FP32 rounding), the scales 2 c / (A w) below and above it.
struct NearPeak {
    float ch, cl, s, sr;
    template <bool SEC>
    __device__ __forceinline__ static NearPeak of(float pt, float ptl, float mu,
                                                  float iw2, float iw2r, float c) {
        const float ch = pt + mu, bb = ch - pt;
        const float e = (pt - (ch - bb)) + (mu - bb);   // exact: pt + mu - ch
        return NearPeak{ch, e + ptl, SEC ? iw2 * c : iw2, SEC ? iw2r * c : iw2r};
    }
    // q2 at the node u of a leaf, relative to its middle m, as the centre is here:
    // an absolute error of a few FP32 roundings of the leaf's extent
    template <bool ASYM>
    __device__ __forceinline__ float q2_node(float u, float m, bool &up) const {
        const float c = (ch - m) + cl;
        if (ASYM) {
            const float d = u - c;
            up = d >= 0.f;
            return d * (up ? sr : s);
        }
        up = false;
        return fmaf(u, s, -c * s);
    }
    // q2 at the point u + ul; whether it lies at or above the centre (SIDE: where
    // the points lie, if known)
    template <bool ASYM, int SIDE = ASYM ? kBoth : kBelow>
    __device__ __forceinline__ float q2(float u, float ul, bool &up) const {
        if (SIDE == kBoth) {
            const float d = (u - ch) + (ul - cl);
            up = d >= 0.f;
            return d * (up ? sr : s);
        }
        up = SIDE == kAbove;
        const float a = up ? sr : s;
        return fmaf(u - ch, a, fmaf(ul, a, -cl * a));
    }
};

// Wave priority in the phase loops, by the phases the wave has left: a wave
// with more of them issues first.  Among waves of one priority the oldest
// issues first, so without this the first waves of a block finish early and
// the last one ends alone, waiting on its own latencies.
__device__ __forceinline__ void prio_left(int left) {
    if (left >= 4) __builtin_amdgcn_s_setprio(3);
    else if (left == 3) __builtin_amdgcn_s_setprio(2);
    else if (left == 2) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// Whether every peak is taken at every point (dense_direct): while T peaks and K
// phases, each a peak's worth or two (twelve sums of an asymmetric one), cost less
// than the stages around the nodes.  A block of four samples, step in us against
// the nodes': N = 3501, S = 64, 60 peaks in one phase 32.2 and 34.4, 80 34.2 and
// 33.8, 8 x 10 36.1 and 36.3, 16 x 5 36.8 and 35.5, asymmetric 8 x 8 39.3 and 40.7,
// 16 x 5 44.6 and 40.1; in five rounds of blocks (N = 7438, S = 100) 80 57.3 and
// 67.2, 128 72.5 and 68.5, asymmetric 16 x 5 83.6 and 80.7.  A block of one sample:
// N = 1500, S = 30, 8 x 16 30.6 and 34.7, 46 x 2 35.7 and 34.3, asymmetric 30 x 3 36.7
// and 36.8.
constexpr int kDirectPhases = 48;
constexpr int direct_most(int SG) { return SG == 1 ? 128 : 88; }
template <int SG, bool ASYM>
__host__ __device__ constexpr bool direct_peaks(int K, int T) {
    return K <= kDirectPhases && T + (ASYM && SG > 1 ? 2 : 1) * K <= direct_most(SG);
}

// Whether the waves share each phase's peaks instead of the phases.
constexpr bool cut_phases(int K) { return 2 * K <= kDenseWaves; }
// Tile t of those of LV leaves; its sums go to place `out` among the
// analysis's tiles.
template <bool GRAD, bool ASYM, bool SEC, int NW, int SG, int LV, bool CUT, typename SM>
__device__ void dense_tile(const ProbDev &P, const StepDev &st, int t, int out, int grp,
                           float *f_out, SM &sm) {
    constexpr bool MID = SM::kMid;
    constexpr int PTS = SM::kPts;
    constexpr int LPS = kWave / SG;         // lanes per sample
    constexpr int PB = kLeaf / LPS;         // points of a leaf per lane
    constexpr int NPP = LV * PB;            // points per lane
    constexpr int SLOTS = LPS / kNodes;     // far peaks taken together
    constexpr int NS = ASYM ? 12 : 6;
    constexpr int NT = NW * kWave;
    constexpr int kCap = SM::kFarCap;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int n = lane % kNodes, sl = lane / LPS, li = lane % LPS, slot = li / kNodes;
    const int S = st.S, K = P.K, s0 = grp * SG;
    const int ns = min(SG, S - s0);
    const int s = s0 + min(sl, ns - 1);     // (lanes past the last sample repeat it)
    const int i0 = t * PTS, i1 = min(i0 + PTS, P.N), np = i1 - i0;
    const int nl = (np + kLeaf - 1) / kLeaf;   // leaves with points
    const double2 mh = mid_half(P, i0, i1);
    const double xref = as_const(P.x)[min(i0 / P.ref * P.ref + P.ref / 2, P.N - 1)];

    // middles and half-widths of the leaves
    double2 h[LV];
#pragma unroll
    for (int l = 0; l < LV; ++l) h[l] = leaf_mid_half(P, i0 + min(l, nl - 1) * kLeaf);
    // The last kPlanPhases threads find the first phases' near ranges (below),
    // the waves before them form the weights: eight those of the leaves' nodes at
    // the points (32 points together), four those of the tile's at the leaves'
    // (and bring in the points).
    constexpr int NC = NT - kPlanPhases, LW = 8;
    static_assert(NW == LW + 4 + kPlanPhases / kWave && PTS <= 4 * kWave, "roles of the waves");
    const double cn = kNodeCos[n];
    if (wv < LW) {
        constexpr int R = LW * (kWave / kNodes), H = kLeaf / R;   // rows a pass, passes a leaf
        const int row = wv * (kWave / kNodes) + lane / kNodes;
        const double num = kNodeNum[n];
        double x[LV * H];
#pragma unroll
        for (int i = 0; i < LV * H; ++i) x[i] = P.x[min(i0 + i * R + row, P.N - 1)];
#pragma unroll
        for (int i = 0; i < LV * H; ++i) {
            const double t = (x[i] - h[i / H].x) * inverse(h[i / H].y);
            sm.lm[(i * R + row) * kNodeStride + n] =
                i * R + row < np ? node_weight(t, cn, num) : 0.f;
        }
    } else if (tid < NC) {
        const int q = tid - LW * kWave, row = q / kNodes;
        const double num = kNodeNum[n], cr = kNodeCos[row], ih = inverse(mh.y);
        const float uq = q < np ? P.u[i0 + q] : 0.f, ulq = q < np ? P.ul[i0 + q] : 0.f;
#pragma unroll
        for (int l = 0; l < LV; ++l)
            sm.em[(l * kNodes + row) * kNodeStride + n] =
                node_weight((h[l].x - mh.x + h[l].y * cr) * ih, cn, num);
        if (q < PTS) {
            sm.us[q] = uq;
            sm.ul[q] = ulq;
        }
    }
    // the lane's nodes, the leaves' relative to their rounded middles; lane n
    // tests the reach of leaf n % LV
    const float vn = (float)((mh.x - xref) + mh.y * cn);
    float vl[LV], lm[LV], lmid = 0.f, lhalf = 0.f;
#pragma unroll
    for (int l = 0; l < LV; ++l) {
        lm[l] = (float)(h[l].x - xref);
        vl[l] = (float)((h[l].x - xref - (double)lm[l]) + h[l].y * cn);
        if (n % LV == l) {
            lmid = lm[l];
            lhalf = (float)h[l].y;
        }
    }

    const float4 *pk = st.pk + (size_t)s * K;
    const float *pkr = ASYM ? st.pkr + (size_t)s * K : nullptr;
    const float4 *sec = SEC ? st.psec + (size_t)s * P.T : nullptr;
    cptr<float> ptt = as_const(P.pt + (size_t)(i0 / P.ref) * P.T);
    cptr<float> ptl = as_const(P.ptl + (size_t)(i0 / P.ref) * P.T);
    cptr<float> inten = as_const(P.inten);
    cptr<int> off = as_const(P.off);

    // The waves take the phases in turn.  With at most half as many phases as
    // waves (CUT) each phase is cut in 2^ps shares, which take the place of phases:
    // share i has the phase i >> ps, and of its near peaks and of those below
    // and above them a part each.  (One wave a phase: K = 1 of 200 peaks, N =
    // 3501, S = 64 took 75 us, K = 2 of 500 137 us; shares of consecutive peaks,
    // of which one has the near ones, K = 2 of 5000 801 us for 260.  A template
    // parameter: the shares' ranges cost the scalar registers of 200 x 60 peaks,
    // S = 128 10 of 699 us.)
    int ps = 0;
    if (CUT)
        while (K << (ps + 1) <= NW) ++ps;
    const int KS = K << ps;
    static_assert(3 * NW <= kPlanPhases, "ranges of the shares");
    // near ranges of the shares [c0, c0 + kPlanPhases); those of cut phases are
    // followed by the ranges below and above
    auto plan = [&](int c0) {
        const int kk = tid - NC;
        if (kk >= 0 && c0 + kk < KS) {
            const int k = (c0 + kk) >> ps;
            const int2 r = dense_near<SEC>(P, st, t, LV, k, s0, ns, mh);
            if (CUT) {
                const auto part = [&](int j0, int j1) {
                    const long long m = max(j1 - j0, 0), q = kk & ((1 << ps) - 1);
                    return make_int2(j0 + (int)(m * q >> ps), j0 + (int)(m * (q + 1) >> ps));
                };
                sm.nr[kk] = part(r.x, r.y);
                sm.nr[NW + kk] = part(P.off[k], r.x);
                sm.nr[2 * NW + kk] = part(r.y, P.off[k + 1]);
            } else {
                sm.nr[kk] = r;
            }
        }
        __syncthreads();
    };
    auto range = [&](int i) {
        const int2 r = sm.nr[i % kPlanPhases];
        return make_int2(__builtin_amdgcn_readfirstlane(r.x),
                         __builtin_amdgcn_readfirstlane(r.y));
    };
    // peaks of share i of a phase with the peaks [a, b)
    struct Peaks {
        int2 near, below, above;
    };
    auto peaks_of = [&](int i, int a, int b) {
        const int2 nr = range(i);
        if (!CUT) return Peaks{nr, make_int2(a, nr.x), make_int2(nr.y, b)};
        return Peaks{nr, range(NW + i), range(2 * NW + i)};
    };
    // the far sums of a phase: lo of the peaks above the tile (its points
    // see their low side), hi of those below
    auto far_of = [&](auto grad, const Peaks &pe, float4 c, float iw2r, float ka,
                      FarSums &lo, FarSums &hi) {
        constexpr bool G = decltype(grad)::value;
        const float um = vn - c.w;
        if (ASYM) {
            hi = far_sums<SLOTS, G, SEC>(ptt, inten, sec, pe.below.x, pe.below.y, slot, um * iw2r,
                                         iw2r, ka);
            lo = far_sums<SLOTS, G, SEC>(ptt, inten, sec, pe.above.x, pe.above.y, slot, um * c.x, c.x,
                                         1.f);
        } else {
            const FarSums x = far_sums<SLOTS, G, SEC>(ptt, inten, sec, pe.below.x, pe.below.y, slot,
                                                      um * c.x, c.x, 1.f);
            const FarSums y = far_sums<SLOTS, G, SEC>(ptt, inten, sec, pe.above.x, pe.above.y, slot,
                                                      um * c.x, c.x, 1.f);
            lo = FarSums{x.f0 + y.f0, x.f1 + y.f1, x.f2 + y.f2};
            hi = FarSums{0.f, 0.f, 0.f};
        }
    };
    // a near peak of the tile, and the reach of its Gaussian; its data are read
    // one peak ahead
    struct Near {
        NearPeak pk;
        float I, c, tw, reach;
    };
    struct NearData {
        float pt, ptl, I;
        float4 rec;
    };
    auto near_data = [&](int j) {
        NearData d{};
        d.pt = ptt[j];
        d.ptl = ptl[j];
        if (SEC) d.rec = sec[j];
        else d.I = inten[j];
        return d;
    };
    auto near_peak = [&](const NearData &d, float4 c, float iw2r) {
        Near r{};
        r.I = SEC ? d.rec.y : d.I;
        r.c = SEC ? d.rec.x : 1.f;
        r.tw = SEC ? d.rec.z : 0.f;
        r.pk = NearPeak::of<SEC>(d.pt, d.ptl, c.w, c.x, iw2r, r.c);
        r.reach = (float)(2.0 * kGaussReach) *
                  rcp_f32(ASYM ? fminf(r.pk.s, r.pk.sr) : r.pk.s);
        return r;
    };
    // Whether the peaks of a phase are taken at the leaves' nodes wherever they
    // lie: those at least kWide half-widths of every leaf wide (for every sample)
    // are as smooth there as one kFarRadius of them away.
    auto wide_phase = [&](float4 c, float iw2r) {
        const float s = ASYM ? fmaxf(c.x, iw2r) : c.x;
        return MID && __builtin_amdgcn_ballot_w64(!(s * lhalf <= (float)(2.0 / kWide))) == 0;
    };
    // The leaves at whose points the peak is taken, one bit each (lane n of a
    // sample tests leaf n mod LV): those that it is near of, or its Gaussian
    // reaches, for some sample; of a wide phase those with the centre of an
    // asymmetric peak, where its width changes.
    auto near_leaves = [&](const Near &r, bool wide) -> unsigned {
        if (wide && !ASYM) return 0;
        const float d = fabsf(r.pk.ch - lmid), far = lhalf + fmaxf(lhalf, r.reach);
        unsigned long long b = __builtin_amdgcn_ballot_w64(!(d >= (wide ? lhalf : far)));
        b |= b >> 32;
        return (unsigned)(b | (b >> 16));
    };

    // the leaves with the centre for some sample
    auto centre_leaves = [&](const Near &r) -> unsigned {
        unsigned long long b = __builtin_amdgcn_ballot_w64(!(fabsf(r.pk.ch - lmid) >= lhalf));
        b |= b >> 32;
        return (unsigned)(b | (b >> 16));
    };

    // ---------------- forward: this wave's phases
    float sig[NPP], lsig[LV], nsig = 0.f, u[NPP], ul[MID ? 1 : NPP];
    // (kept in registers where there are few)
    auto ul_of = [&](int p) { return MID ? sm.ul[p * LPS + li] : ul[p]; };
#pragma unroll
    for (int p = 0; p < NPP; ++p) sig[p] = 0.f;
#pragma unroll
    for (int l = 0; l < LV; ++l) lsig[l] = 0.f;
    for (int c0 = 0; c0 < KS; c0 += kPlanPhases) {
        if (c0 > 0) __syncthreads();
        plan(c0);
        if (c0 == 0) {
#pragma unroll
            for (int p = 0; p < NPP; ++p) {
                u[p] = sm.us[p * LPS + li];
                if (!MID) ul[p] = sm.ul[p * LPS + li];
            }
        }
        for (int i = c0 + wv; i < min(KS, c0 + kPlanPhases); i += NW) {
            prio_left((min(KS, c0 + kPlanPhases) - i + NW - 1) / NW);
            const int k = i >> ps, a = off[k], b = off[k + 1];
            if (a >= b) continue;
            const Peaks pe = peaks_of(i, a, b);
            const float4 c = pk[k];
            const float iw2r = ASYM ? pkr[k] : c.x;
            const float ka = ASYM && SEC ? c.x / iw2r : 1.f;   // alpha
            FarSums lo, hi;
            if (GRAD && i < kCap) {
                far_of(std::true_type{}, pe, c, iw2r, ka, lo, hi);
                float (*dst)[kWave] = sm.far[i];
                constexpr int H = SM::kFarSums / 2;   // (ASYM: the high side)
                dst[0][lane] = lo.f0; dst[1][lane] = lo.f1; dst[2][lane] = lo.f2;
                if (ASYM) {
                    dst[H][lane] = hi.f0; dst[H + 1][lane] = hi.f1; dst[H + 2][lane] = hi.f2;
                }
            } else {
                far_of(std::false_type{}, pe, c, iw2r, ka, lo, hi);
            }
            nsig = fmaf(c.z, lo.f0 + hi.f0, nsig);
            const bool wide = wide_phase(c, iw2r);
            NearData next = near_data(min(pe.near.x, b - 1));
            for (int j = pe.near.x; j < pe.near.y; ++j) {
                const Near r = near_peak(next, c, iw2r);
                next = near_data(min(j + 1, b - 1));
                const float aL = c.z * r.I, aG = c.y * r.I;
                auto at_point = [&](int p) {
                    bool up;
                    const float q2 = r.pk.template q2<ASYM>(u[p], ul_of(p), up);
                    const float tt = fmaf(q2, q2, 1.0f);
                    sig[p] = fmaf(aL, rcp_f32(tt), sig[p]);
                    sig[p] = fmaf(aG, exp2_f32(-tt), sig[p]);
                };
                if constexpr (!MID) {
                    // (no branches: bound by latency)
#pragma unroll
                    for (int p = 0; p < NPP; ++p) at_point(p);
                    continue;
                }
                const unsigned near = near_leaves(r, wide);
#pragma unroll
                for (int l = 0; l < LV; ++l) {
                    if (l >= nl) break;
                    if (near >> l & 1u) {
                        asm volatile("");    // (a branch, not selects)
#pragma unroll
                        for (int q = 0; q < PB; ++q) at_point(l * PB + q);
                    } else {
                        asm volatile("");
                        bool up;
                        const float q2 = r.pk.template q2_node<ASYM>(vl[l], lm[l], up);
                        const float tt = fmaf(q2, q2, 1.0f);
                        lsig[l] = fmaf(aL, rcp_f32(tt), lsig[l]);
                        if (wide) {
                            asm volatile("");
                            lsig[l] = fmaf(aG, exp2_f32(-tt), lsig[l]);
                        }
                    }
                }
            }
        }
    }
    __builtin_amdgcn_s_setprio(3);
#pragma unroll
    for (int p = 0; p < NPP; ++p) sm.sig[wv][sl][p * LPS + li] = sig[p];
    sm.nod[wv][lane] = nsig;
    if (MID) {
#pragma unroll
        for (int l = 0; l < LV; ++l) sm.ndl[wv][l][lane] = lsig[l];
    }
    // (the point stage's loads go out before the waves meet)
    static_assert(NT % PTS == 0, "a thread's points share their index in the tile");
    double py = 0.0, pb = 0.0, pl = 0.0;
    {
        const int i = min(i0 + tid % PTS, P.N - 1);
        py = P.y[i];
        pb = P.bg[i];
        pl = P.lgy[i];
    }
    __syncthreads();
    // node sums over the waves, the tile's then brought to the leaves': the
    // lanes of a group of NG take the terms of one sum
    {
        constexpr int NG = NT / (SG * kNodes) < 64 ? NT / (SG * kNodes) : 64;
        const int o = tid / NG, j = tid % NG;
        if (o < SG * kNodes) {
            const int g = o / kNodes, m = o % kNodes;
            double v = 0.0;
            for (int x = j; x < NW * SLOTS; x += NG)
                v += (double)sm.nod[x / SLOTS][g * LPS + x % SLOTS * kNodes + m];
#pragma unroll
            for (int x = NG / 2; x >= 1; x >>= 1) v += __shfl_xor(v, x, kWave);
            if (j == 0) sm.pn[g][m] = v;
        }
    }
    __syncthreads();
    {
        constexpr int OUT = SG * SM::kLow;
        constexpr int NG = NT / OUT < 16 ? NT / OUT : 16;
        static_assert(OUT * NG <= NT, "one pass");
        const int o = tid / NG, j = tid % NG;
        if (o < OUT) {
            const int g = o / SM::kLow, q = o % SM::kLow;
            double v = 0.0;
            if (MID)
#pragma unroll
                for (int w = j; w < NW; w += NG)
                    v += (double)sm.ndl[w][q / kNodes][g * kNodes + q % kNodes];
#pragma unroll
            for (int m = j; m < kNodes; m += NG)
                v = fma((double)sm.em[q * kNodeStride + m], sm.pn[g][m], v);
#pragma unroll
            for (int x = NG / 2; x >= 1; x >>= 1) v += __shfl_xor(v, x, kWave);
            if (j == 0) sm.low[g][q] = v;
        }
    }
    __syncthreads();

    // ---------------- points: f = B + near + interpolated far sums (FP64),
    // the Poisson log-likelihood and the residual
    for (int q = tid; q < SG * PTS; q += NT) {
        const int g = q / PTS, qq = q % PTS, i = i0 + qq, ss = s0 + g;
        double ll = 0.0;
        float rr = 0.f;
        if (i < P.N && ss < S) {
            const double *low = sm.low[g] + qq / kLeaf * kNodes;
            double sg = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) sg += (double)sm.sig[w][g][qq];
#pragma unroll
            for (int m = 0; m < kNodes; ++m)
                sg = fma((double)sm.lm[qq * kNodeStride + m], low[m], sg);
            const double f = pb + sg, y = py;   // (PTS divides NT: one point per thread)
            if (f_out) f_out[(size_t)ss * P.N + i] = (float)f;
            if (GRAD || st.llp) {
                if (st.llp) ll = (y != 0.0 ? y * log(f) : 0.0) - f - pl;
                rr = (float)(y / f - 1.0);
            }
        }
        sm.rres[g][qq] = rr;
        ll = wave_sum(ll);
        if (lane == 0) sm.red[q / kWave] = ll;
    }
    __syncthreads();
    if (tid < ns && st.llp) {
        double v = 0.0;
#pragma unroll
        for (int l = 0; l < LV; ++l) v += sm.red[tid * LV + l];
        st.llp[(size_t)(s0 + tid) * st.nt + out] = v;
    }
    if (!GRAD) return;

    // ---------------- the residual at the leaves' nodes, then at the tile's
    {
        constexpr int OUT = SG * SM::kLow;
        constexpr int TPO = NT / OUT < kWave ? NT / OUT : kWave;
        const int o = tid / TPO, j = tid % TPO;
        if (o < OUT) {
            const int g = o / SM::kLow, m = o % SM::kLow, q0 = m / kNodes * kLeaf;
            double v = 0.0;
            if (m / kNodes < nl)
#pragma unroll 4
                for (int q = q0 + j; q < q0 + kLeaf; q += TPO)
                    v = fma((double)sm.lm[q * kNodeStride + m % kNodes], (double)sm.rres[g][q],
                            v);
#pragma unroll
            for (int x = TPO / 2; x >= 1; x >>= 1) v += __shfl_xor(v, x, kWave);
            if (j == 0) sm.low[g][m] = v;
        }
    }
    __syncthreads();
    {
        constexpr int NG = NT / (SG * kNodes) < 64 ? NT / (SG * kNodes) : 64;
        const int o = tid / NG, j = tid % NG;
        if (o < SG * kNodes) {
            const int g = o / kNodes, m = o % kNodes;
            double v = 0.0;
            for (int q = j; q < nl * kNodes; q += NG)
                v = fma((double)sm.em[q * kNodeStride + m], sm.low[g][q], v);
#pragma unroll
            for (int x = NG / 2; x >= 1; x >>= 1) v += __shfl_xor(v, x, kWave);
            if (j == 0) sm.rn[g][m] = v;
        }
    }
    __syncthreads();

    // ---------------- adjoint: the phase's sums over points and nodes
    const float rn = (float)sm.rn[sl][n];
    float r[NPP], rl[LV];
#pragma unroll
    for (int p = 0; p < NPP; ++p) r[p] = sm.rres[sl][p * LPS + li];
#pragma unroll
    for (int l = 0; l < LV; ++l) rl[l] = MID ? (float)sm.low[sl][l * kNodes + n] : 0.f;
    for (int c0 = 0; c0 < KS; c0 += kPlanPhases) {
        if (K > kPlanPhases) {          // (otherwise the ranges are still there)
            __syncthreads();
            plan(c0);
        }
        for (int i = c0 + wv; i < min(KS, c0 + kPlanPhases); i += NW) {
            prio_left((min(KS, c0 + kPlanPhases) - i + NW - 1) / NW);
            const int k = i >> ps, a = off[k], b = off[k + 1];
            float acc[NS];
#pragma unroll
            for (int q = 0; q < NS; ++q) acc[q] = 0.f;
            if (a < b) {
                const Peaks pe = peaks_of(i, a, b);
                const float4 c = pk[k];
                const float iw2r = ASYM ? pkr[k] : c.x;
                const float ka = ASYM && SEC ? c.x / iw2r : 1.f;
                FarSums lo, hi{0.f, 0.f, 0.f};
                if (i < kCap) {
                    float (*src)[kWave] = sm.far[i];
                    constexpr int H = SM::kFarSums / 2;
                    lo = FarSums{src[0][lane], src[1][lane], src[2][lane]};
                    if (ASYM) hi = FarSums{src[H][lane], src[H + 1][lane], src[H + 2][lane]};
                } else {
                    far_of(std::true_type{}, pe, c, iw2r, ka, lo, hi);
                }
                acc[3] = rn * lo.f0; acc[4] = rn * lo.f1; acc[5] = rn * lo.f2;
                if constexpr (ASYM) {
                    acc[9] = rn * hi.f0; acc[10] = rn * hi.f1; acc[11] = rn * hi.f2;
                }
                const bool wide = wide_phase(c, iw2r);
                NearData next = near_data(min(pe.near.x, b - 1));
                for (int j = pe.near.x; j < pe.near.y; ++j) {
                    const Near rec = near_peak(next, c, iw2r);
                    next = near_data(min(j + 1, b - 1));
                    const SecW wl = SecW::of(rec.tw), wh = SecW::of(rec.tw * ka);
                    // the peak's own sums, its intensity applied at the end
                    float e[NS];
#pragma unroll
                    for (int q = 0; q < NS; ++q) e[q] = 0.f;
                    auto at_point = [&](int p) {
                        bool up;
                        const float q2 = rec.pk.template q2<ASYM>(u[p], ul_of(p), up);
                        const float tt = fmaf(q2, q2, 1.0f);
                        adj_terms_L<ASYM, SEC>(r[p], q2, tt, up, rec.c, wl, wh, e);
                        adj_point_G<ASYM, SEC>(AdjPt{r[p], q2, tt, up}, rec.c, wl, wh, e);
                    };
                    // a leaf without the centre of an asymmetric peak: the lane's
                    // points lie on one side of it, and the sums are put there once
                    const unsigned inside = ASYM ? centre_leaves(rec) : 0u;
                    auto one_side = [&](int l) {
                        const bool up = lm[l] >= rec.pk.ch;
                        const float s1 = up ? rec.pk.sr : rec.pk.s;
                        float h[NS];
#pragma unroll
                        for (int q = 0; q < 6; ++q) h[q] = 0.f;
#pragma unroll
                        for (int q = 0; q < PB; ++q) {
                            const int p = l * PB + q;
                            const float q2 = ((u[p] - rec.pk.ch) + (ul_of(p) - rec.pk.cl)) * s1;
                            const float tt = fmaf(q2, q2, 1.0f);
                            adj_terms_L<ASYM, SEC, kBelow>(r[p], q2, tt, up, rec.c, wl, wh, h);
                            adj_point_G<ASYM, SEC, kBelow>(AdjPt{r[p], q2, tt, up}, rec.c, wl,
                                                           wh, h);
                        }
                        const float fu = up ? 1.f : 0.f, fd = 1.f - fu;
#pragma unroll
                        for (int q = 0; q < 6; ++q) {
                            e[q] = fmaf(fd, h[q], e[q]);
                            if constexpr (ASYM) e[6 + q] = fmaf(fu, h[q], e[6 + q]);
                        }
                    };
                    if constexpr (!MID) {
#pragma unroll
                        for (int p = 0; p < NPP; ++p) at_point(p);
                    } else {
                        const unsigned near = near_leaves(rec, wide);
#pragma unroll
                        for (int l = 0; l < LV; ++l) {
                            if (l >= nl) break;
                            if (ASYM && (near & ~inside) >> l & 1u) {
                                asm volatile("");
                                one_side(l);
                            } else if (near >> l & 1u) {
                                asm volatile("");
#pragma unroll
                                for (int q = 0; q < PB; ++q) at_point(l * PB + q);
                            } else {
                                asm volatile("");
                                bool up;
                                const float q2 =
                                    rec.pk.template q2_node<ASYM>(vl[l], lm[l], up);
                                const float tt = fmaf(q2, q2, 1.0f);
                                adj_terms_L<ASYM, SEC>(rl[l], q2, tt, up, rec.c, wl, wh, e);
                                if (wide) {
                                    asm volatile("");
                                    adj_point_G<ASYM, SEC>(AdjPt{rl[l], q2, tt, up}, rec.c, wl,
                                                           wh, e);
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int q = 0; q < NS; ++q) acc[q] = fmaf(rec.I, e[q], acc[q]);
                }
            }
#pragma unroll
            for (int q = 0; q < NS; ++q) acc[q] = lanes_total<LPS>(acc[q]);
            // (a row of 16 lanes holds the totals: lane q of it stores sum q)
            float v = acc[0];
#pragma unroll
            for (int q = 1; q < NS; ++q) v = n == q ? acc[q] : v;
            if (n < NS && slot == SLOTS - 1 && sl < ns) {
                if (CUT) sm.nod[i][sl * NS + n] = v;
                else st.part[(((size_t)out * K + k) * S + s) * NS + n] = v;
            }
        }
    }
    if (CUT) {
        // the phases' sums over their shares
        static_assert(SG * NS <= kWave + 1, "a share's sums fit its row");
        __syncthreads();
        for (int i = tid; i < K * ns * NS; i += NT) {
            const int k = i / (ns * NS), q = i % (ns * NS);
            double v = 0.0;
            for (int w = k << ps; w < (k + 1) << ps; ++w) v += (double)sm.nod[w][q];
            st.part[(((size_t)out * K + k) * S + s0) * NS + q] = (float)v;
        }
    }
}

// ---- few peaks: every one at every point --------------------------------------
//
// Around the phase loops a block of dense_tile spends some 10 us on weights,
// ranges and nodes, which few peaks do not earn back.  Here the peaks of the
// block's samples are prepared in LDS by a thread each; then the waves take a
// sample, a share of its peaks and (with four samples) all leaves each: the sum
// over the peaks, the likelihood, then the adjoint terms of the share's phases,
// reduced over the wave and added over the waves.  A lane with a point of each
// leaf reads a peak once for them, and skips the Gaussian and the side of an
// asymmetric peak that none of the tile's points has.  (With one point per lane,
// peaks dealt out one by one and six totals apart: 4 x 8 peaks, N = 13620, S = 79
// 74 us a step for 57, asymmetric 5 x 7, N = 7438, S = 100 89 for 60; four-wave
// blocks of one sample at every point 67 and 75.)  Bound by issue in many rounds of
// blocks, by latency below.  The same tiles and places as dense_tile's.

// Totals over the wave of NS (6 or 12) values, that of value q in lane q: pairs of
// values are packed as lanes are added (about half the instructions of NS totals,
// which with few peaks a phase are a third of the adjoint).
template <int NS>
__device__ __forceinline__ float wave_totals(const float (&e)[NS], int lane) {
    const bool b0 = lane & 1, b1 = lane & 2;
    float f[NS / 2];
#pragma unroll
    for (int i = 0; i < NS / 2; ++i) {
        const float keep = b0 ? e[2 * i + 1] : e[2 * i], give = b0 ? e[2 * i] : e[2 * i + 1];
        f[i] = keep + dpp_f32<0xB1, 0xf, true>(give);       // lane ^ 1
    }
    constexpr int NG = (NS / 2 + 1) / 2;
    float r = 0.f;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        float g;
        if (2 * i + 1 < NS / 2) {
            const float keep = b1 ? f[2 * i + 1] : f[2 * i], give = b1 ? f[2 * i] : f[2 * i + 1];
            g = keep + dpp_f32<0x4E, 0xf, true>(give);      // lane ^ 2
        } else {
            g = f[2 * i] + dpp_f32<0x4E, 0xf, true>(f[2 * i]);
        }
        g += dpp_f32<0x124, 0xf, true>(g);                  // row_ror:4
        g += dpp_f32<0x128, 0xf, true>(g);                  // row_ror:8
        const auto s16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(g), __float_as_uint(g),
                                                          false, false);
        g = __uint_as_float(s16[0]) + __uint_as_float(s16[1]);      // rows in pairs
        const auto s32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(g), __float_as_uint(g),
                                                          false, false);
        g = __uint_as_float(s32[0]) + __uint_as_float(s32[1]);
        r = lane >> 2 == i ? g : r;
    }
    return r;
}

template <int NW, int SG, int LV, bool ASYM>
struct DirectSmem {
    static constexpr int kPts = LV * kLeaf, kMost = direct_most(SG);
    static constexpr int kLane = SG == 1 ? 1 : LV;      // points of a lane
    static constexpr int kShares = NW * kLane / (SG * LV);
    float4 at[SG][kMost];                 // NearPeak
    float4 amp[SG][kMost];                // (aL, aG, I, c) ...
    float tw[SG][kMost];
    int kind[SG][kMost];                  // bit 0: the Gaussian reaches the tile,
                                          // 1, 2: all points above, below the centre
    float rres[SG * kPts];                // residual y/f - 1
    double red[SG * LV];
    union {
        double sig[kShares][SG * kPts];                     // the shares' sums at the points,
        float acc[kDirectPhases][NW][ASYM ? 12 : 6];        // then the waves' adjoint sums
    };
};

template <bool GRAD, bool ASYM, bool SEC, int NW, int SG, int LV, typename SM>
__device__ void dense_direct(const ProbDev &P, const StepDev &st, int t, int out, int grp,
                             float *f_out, SM &sm) {
    constexpr int PTS = LV * kLeaf, NT = NW * kWave, SH = SM::kShares;
    constexpr int PP = SM::kLane, LG = LV / PP;
    constexpr int NS = ASYM ? 12 : 6;
    static_assert(SH * SG * PTS == NT * PP, "PP points per share, sample and thread");
    static_assert(SM::kMost <= 2 * kWave, "two words of kinds");
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int S = st.S, K = P.K, T = P.T, s0 = grp * SG, ns = min(SG, S - s0);
    const int i0 = t * PTS;
    // the wave's share, sample and leaves of the sums
    const int sh = wv / (SG * LG), g = wv / LG % SG, p0 = wv % LG * (PP * kLeaf) + lane;
    const int ja = T * sh / SH, jb = T * (sh + 1) / SH;      // the share's peaks
    const int gs = min(g, ns - 1);       // (waves past the last sample repeat it)
    float u[PP], ul[PP];
#pragma unroll
    for (int p = 0; p < PP; ++p) {
        const int ic = min(i0 + p0 + p * kLeaf, P.N - 1);
        u[p] = P.u[ic];
        ul[p] = P.ul[ic];
    }
    // the thread's sample and point of the likelihood
    const int gq = tid % (SG * PTS), gl = gq / PTS, i = i0 + gq % PTS, ic = min(i, P.N - 1);
    const bool in = i < P.N && gl < ns;
    const double py = P.y[ic], pb = P.bg[ic], pl = P.lgy[ic];
    cptr<int> off = as_const(P.off);
    const float ua = P.u[i0], ub = P.u[min(i0 + PTS, P.N) - 1];
    for (int x = tid; x < ns * T; x += NT) {
        const int gg = x / T, j = x % T, k = P.phase[j], s = s0 + gg;
        const float4 c = st.pk[(size_t)s * K + k];
        const float iw2r = ASYM ? st.pkr[(size_t)s * K + k] : c.x;
        const float4 r = SEC ? st.psec[(size_t)s * T + j] : make_float4(1.f, P.inten[j], 0.f, 0.f);
        const size_t o = (size_t)(i0 / P.ref) * T + j;
        const NearPeak p = NearPeak::of<SEC>(P.pt[o], P.ptl[o], c.w, c.x, iw2r, r.x);
        sm.at[gg][j] = make_float4(p.ch, p.cl, p.s, p.sr);
        sm.amp[gg][j] = make_float4(c.z * r.y, c.y * r.y, r.y, r.x);
        if (SEC) sm.tw[gg][j] = r.z;
        constexpr float kOut = (float)(2.0 * kGaussReach), kClear = 1e-3f;
        const float da = ua - p.ch, db = p.ch - ub;
        if (PP > 1)
            sm.kind[gg][j] = (da * p.sr > kOut || db * p.s > kOut ? 0 : 1) |
                             (da > kClear ? 2 : 0) | (db > kClear ? 4 : 0);
    }
    __syncthreads();
    // the peaks' kinds, a bit each
    uint64_t kinds[3][2];
#pragma unroll
    for (int b = 0; b < (PP > 1 ? (ASYM ? 3 : 1) : 0); ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = lane + h * kWave;
            kinds[b][h] = __builtin_amdgcn_ballot_w64(j < T && (sm.kind[gs][j] >> b & 1));
        }
    auto is_kind = [&](int b, int j) {
        return (kinds[b][j >= kWave] >> (j & (kWave - 1)) & 1) != 0;
    };
    auto reaches = [&](int j) { return PP == 1 || is_kind(0, j); };
    auto peak_of = [&](int j) {
        const float4 a = sm.at[gs][j];
        return NearPeak{a.x, a.y, a.z, a.w};
    };
    // (four peaks in FP32, their sums in FP64)
    double sum[PP];
#pragma unroll
    for (int p = 0; p < PP; ++p) sum[p] = 0.0;
    auto value = [&](int j, float *v) {
        const NearPeak pk = peak_of(j);
        const float4 m = sm.amp[gs][j];
        float tt[PP];
#pragma unroll
        for (int p = 0; p < PP; ++p) {
            bool up;
            const float q2 = pk.template q2<ASYM>(u[p], ul[p], up);
            tt[p] = fmaf(q2, q2, 1.0f);
            v[p] = fmaf(m.x, rcp_f32(tt[p]), v[p]);
        }
        if (reaches(j)) {
            if (PP > 1) asm volatile("");    // (a branch, not selects)
#pragma unroll
            for (int p = 0; p < PP; ++p) v[p] = fmaf(m.y, exp2_f32(-tt[p]), v[p]);
        }
    };
    auto values = [&](int j, int n) {
        float v[PP];
#pragma unroll
        for (int p = 0; p < PP; ++p) v[p] = 0.f;
#pragma unroll
        for (int x = 0; x < n; ++x) value(j + x, v);
#pragma unroll
        for (int p = 0; p < PP; ++p) sum[p] += (double)v[p];
    };
    int j = ja;
    for (; j + 4 <= jb; j += 4) values(j, 4);
    for (; j < jb; ++j) values(j, 1);
    if (SH > 1) {
#pragma unroll
        for (int p = 0; p < PP; ++p) sm.sig[sh][g * PTS + p0 + p * kLeaf] = sum[p];
        __syncthreads();
    }
    if (tid < SG * PTS) {
        double sg = SH > 1 ? sm.sig[0][gq] : sum[0];
#pragma unroll
        for (int x = 1; x < SH; ++x) sg += sm.sig[x][gq];
        const double f = pb + sg;
        if (in && f_out) f_out[(size_t)(s0 + gl) * P.N + i] = (float)f;
        double ll = in && st.llp ? (py != 0.0 ? py * log(f) : 0.0) - f - pl : 0.0;
        if (GRAD) sm.rres[gq] = in ? (float)(py / f - 1.0) : 0.f;
        ll = wave_sum(ll);
        if (lane == 0) sm.red[wv] = ll;
    }
    __syncthreads();
    if (tid < ns && st.llp) {
        double v = 0.0;
#pragma unroll
        for (int l = 0; l < LV; ++l) v += sm.red[tid * LV + l];
        st.llp[(size_t)(s0 + tid) * st.nt + out] = v;
    }
    if (!GRAD) return;
    float R[PP];
#pragma unroll
    for (int p = 0; p < PP; ++p) R[p] = sm.rres[g * PTS + p0 + p * kLeaf];
    for (int k = 0; k < K; ++k) {
        const int a = max(off[k], ja), b = min(off[k + 1], jb);
        if (a >= b) {                // none of the phase's peaks in the share
            if (lane < NS) sm.acc[k][wv][lane] = 0.f;
            continue;
        }
        float ka = 1.f;
        if (ASYM && SEC) {
            const size_t o = (size_t)(s0 + gs) * K + k;
            ka = st.pk[o].x / st.pkr[o];
        }
        float e[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) e[q] = 0.f;
        auto terms = [&](int j, auto side) {
            constexpr int SIDE = decltype(side)::value;
            const NearPeak pk = peak_of(j);
            const float4 m = sm.amp[gs][j];
            const float tw = SEC ? sm.tw[gs][j] : 0.f;
            const SecW wl = SecW::of(tw), wh = SecW::of(tw * ka);
            float q2[PP], tt[PP];
            bool up[PP];
#pragma unroll
            for (int p = 0; p < PP; ++p) {
                q2[p] = pk.template q2<ASYM, SIDE>(u[p], ul[p], up[p]);
                tt[p] = fmaf(q2[p], q2[p], 1.0f);
                adj_terms_L<ASYM, SEC, SIDE>(R[p] * m.z, q2[p], tt[p], up[p], m.w, wl, wh, e);
            }
            if (reaches(j)) {
                if (PP > 1) asm volatile("");    // (a branch, not selects)
#pragma unroll
                for (int p = 0; p < PP; ++p)
                    adj_point_G<ASYM, SEC, SIDE>(AdjPt{R[p] * m.z, q2[p], tt[p], up[p]}, m.w, wl,
                                                 wh, e);
            }
        };
        using Below = std::integral_constant<int, kBelow>;
        using Above = std::integral_constant<int, kAbove>;
        using Both = std::integral_constant<int, ASYM ? kBoth : kBelow>;
        constexpr int U = PP == 1 ? 4 : 1;
#pragma unroll U
        for (int j = a; j < b; ++j) {
            if (ASYM && PP > 1 && is_kind(1, j)) terms(j, Above{});
            else if (ASYM && PP > 1 && is_kind(2, j)) terms(j, Below{});
            else terms(j, Both{});
        }
        const float v = wave_totals<NS>(e, lane);
        if (lane < NS) sm.acc[k][wv][lane] = v;
    }
    __syncthreads();
    for (int x = tid; x < K * ns * NS; x += NT) {
        const int k = x / (ns * NS), q = x % NS, gg = x / NS % ns;
        double v = 0.0;
        for (int w = 0; w < NW; ++w)
            if (w / LG % SG == gg) v += (double)sm.acc[k][w][q];
        st.part[(((size_t)out * K + k) * S + s0 + gg) * NS + q] = (float)v;
    }
}

}  // namespace xrdvi
