// Background estimation before the analysis (App. A.2: the background is
// estimated beforehand by an iterative least-squares method): asymmetric
// least squares (Eilers and Boelens, 2005).  Repeatedly solve
//     (W + lambda D^T D) z = W y,   D the second-difference operator,
// and set w_i = p where y_i > z_i and 1 - p elsewhere (w = 1 at the start),
// so that the smooth curve z hugs the data from below.
//
// The system A z = r is symmetric positive definite and pentadiagonal.  One
// block per spectrum solves it in parallel by a symmetric reordering: the rows
// split into P interior blocks, a thread each, separated by 2-row separators
// (with bandwidth 2, removing two consecutive rows decouples the blocks).
//  1. Each thread factors its block A_p = L D L^T and, in the same forward
//     sweep, forms the corner 2 x 2 blocks of A_p^{-1} that couple it to its
//     separators, (A_p^{-1})_{ab} = sum_i (L^{-1})_{ia} (L^{-1})_{ib} / d_i, and
//     the corresponding entries of A_p^{-1} r_p.
//  2. The Schur complement on the separators, a block tridiagonal SPD system
//     of 2 x 2 blocks: a thread per separator forms its blocks and solves it by
//     parallel cyclic reduction (log2 P steps, each a Schur complement of every
//     other row's block, so the blocks stay SPD).
//  3. Each thread solves its block with the separator values moved to the
//     right-hand side.
// Every step is elimination without pivoting on a symmetric reordering of
// an SPD matrix, the stable case.  FP64 throughout.
//
// The time is a chain of latencies: per reweighting about N / P rows of a
// pivot's reciprocal each, then log2 P reduction steps.  So P is as large as
// one wave per SIMD (256 threads) holds, or two for long spectra (one wave has
// all blocks of a short one), and a block's rows (pivots, factors, counts) stay in registers from one
// reweighting to the next.  15 reweightings of 3501 points (11 or 12 rows a
// thread): 127 us, of 12 000 355 us (1810 and 5040 us with one wave per spectrum, one
// lane of which eliminated the 63 separators).
#include <cmath>
#include <string>

#include "xrdvi.h"
#include "xrdvi_internal.h"

namespace xrdvi {

namespace {

constexpr int kMinRows = 8;       // interior rows per block, at least

// Entries of D^T D, D the (N-2) x N second-difference matrix with rows
// (1, -2, 1): the diagonal and the first off-diagonal (i, i + 1); the second
// one is 1 everywhere (N >= 3).
__device__ __forceinline__ double dtd0(int i, int N) {
    return (i <= N - 3 ? 1.0 : 0.0) + (i >= 1 && i <= N - 2 ? 4.0 : 0.0) + (i >= 2 ? 1.0 : 0.0);
}
__device__ __forceinline__ double dtd1(int i, int N) {
    return (i <= N - 3 ? -2.0 : 0.0) + (i >= 1 ? -2.0 : 0.0);
}

// 1 / d to a rounding or two (d > 0, normal).
__device__ __forceinline__ double recip(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    return fma(fma(-d, r, 1.0), r, r);
}

struct M2 {
    double a, b, c, d;     // [[a, b], [c, d]]
};
__device__ __forceinline__ M2 mul(const M2 &x, const M2 &y) {
    return M2{x.a * y.a + x.b * y.c, x.a * y.b + x.b * y.d,
              x.c * y.a + x.d * y.c, x.c * y.b + x.d * y.d};
}
__device__ __forceinline__ M2 tr(const M2 &x) { return M2{x.a, x.c, x.b, x.d}; }
__device__ __forceinline__ M2 sub(const M2 &x, const M2 &y) {
    return M2{x.a - y.a, x.b - y.b, x.c - y.c, x.d - y.d};
}
__device__ __forceinline__ M2 neg(const M2 &x) { return M2{-x.a, -x.b, -x.c, -x.d}; }
__device__ __forceinline__ M2 inv_sym(const M2 &x) {
    const double r = recip(x.a * x.d - x.b * x.b);
    return M2{x.d * r, -x.b * r, -x.b * r, x.a * r};
}
__device__ __forceinline__ double2 mulv(const M2 &x, double2 v) {
    return make_double2(x.a * v.x + x.b * v.y, x.c * v.x + x.d * v.y);
}
__device__ __forceinline__ double2 subv(double2 x, double2 y) {
    return make_double2(x.x - y.x, x.y - y.y);
}

// What a block tells the separator before it.
struct BlockLow {
    M2 tl, trr;            // corners of A_p^{-1}: top-left, top-right
    double2 xf;            // first two entries of A_p^{-1} r_p
};
// One row of the separators' system during the reduction.
struct SepRow {
    M2 di, up;             // inverse diagonal block, coupling to the next
    double2 y;
};

// A block's rows: in registers (R > 0; the counts too if Y), else in the
// caller's scratch, row i of all T threads together.  y counts, di inverse
// pivots, l = L_{i,i-1}, u = the forward sweep's values and then z; hit: y_i >
// z_i of the last solution.
template <int T, int R, bool Y>
struct Rows {
    double y_[Y ? R : 1], di_[R], l_[R], u_[R];
    const double *yg_;
    unsigned hit_ = 0;
    __device__ void bind(const double *yg, double *, size_t, int n) {
        yg_ = yg;
        if (Y) {
#pragma unroll
            for (int i = 0; i < R; ++i) y_[i] = i < n ? yg[i] : 0.0;
        }
    }
    __device__ double y(int i) const { return Y ? y_[i] : yg_[i]; }
    __device__ double &di(int i) { return di_[i]; }
    __device__ double &l(int i) { return l_[i]; }
    __device__ double &u(int i) { return u_[i]; }
    __device__ bool hit(int i) const { return hit_ >> i & 1u; }
    __device__ void set_z(int i, double z) {
        hit_ = (hit_ & ~(1u << i)) | (unsigned)(y(i) > z) << i;
    }
};
template <int T, bool Y>
struct Rows<T, 0, Y> {
    // (T n of the longest block <= N - T + 2: it fits the spectrum's share)
    double *y_, *di_, *l_, *u_;
    __device__ void bind(const double *yg, double *scratch, size_t bn, int n) {
        y_ = scratch + threadIdx.x;
        di_ = y_ + bn;
        l_ = di_ + bn;
        u_ = l_ + bn;
        for (int i = 0; i < n; ++i) y_[i * T] = yg[i];
    }
    __device__ double y(int i) const { return y_[i * T]; }
    __device__ double &di(int i) { return di_[i * T]; }
    __device__ double &l(int i) { return l_[i * T]; }
    __device__ double &u(int i) { return u_[i * T]; }
    __device__ bool hit(int i) const { return y_[i * T] > u_[i * T]; }
    __device__ void set_z(int i, double z) { u_[i * T] = z; }
};

// f(i) for i = 0 .. n - 1 (or down), unrolled when the rows are in registers.
template <int R, typename F>
__device__ __forceinline__ void each_row(int n, F f) {
    if constexpr (R > 0) {
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (i < n) f(i);
    } else {
        for (int i = 0; i < n; ++i) f(i);
    }
}
template <int R, typename F>
__device__ __forceinline__ void each_row_down(int n, F f) {
    if constexpr (R > 0) {
#pragma unroll
        for (int i = R - 1; i >= 0; --i)
            if (i < n) f(i);
    } else {
        for (int i = n - 1; i >= 0; --i) f(i);
    }
}

// One block of T threads per spectrum, n_iter reweighting iterations; scratch
// (R = 0 only): four arrays [B][N].
template <int T, int R, bool Y>
__global__ __launch_bounds__(T) void k_asls(int N, const double *__restrict__ y,
                                            double *scratch, double *z, double lambda,
                                            double p, int n_iter) {
    __shared__ BlockLow low_s[T];
    __shared__ SepRow sep_s[2][T];
    __shared__ double2 zs_s[T];
    const int t = threadIdx.x;
    const size_t o = (size_t)blockIdx.x * N;
    const double *yb = y + o;
    double *zb = z + o;
    if (N < 3) {                       // no second differences: z = y
        if (t < N) zb[t] = yb[t];
        return;
    }
    // P blocks share the N - 2 (P - 1) interior rows as evenly as possible
    const int P = max(1, min(T, (N + 2) / (kMinRows + 2))), M = P - 1;
    const int base = (N - 2 * M) / P, extra = (N - 2 * M) % P;
    const int r0 = t * (base + 2) + min(t, extra), n = t < P ? base + (t < extra ? 1 : 0) : 0;
    const int e = r0 + n;              // the separator after this block: rows e, e + 1
    const bool sep = t < M;
    Rows<T, R, Y> rows;
    if (n > 0) rows.bind(yb + r0, scratch + o, (size_t)gridDim.x * N, n);
    const double ys0 = sep ? yb[e] : 0.0, ys1 = sep ? yb[e + 1] : 0.0;
    bool hs0 = false, hs1 = false;
    // couplings of the block's first two rows to the separator before it, of
    // its last two rows to the separator after it, and of the next block's
    // first two rows to that one
    const double c1e = lambda * dtd1(e - 1, N), c1n = lambda * dtd1(e + 1, N);
    const M2 CLt{lambda, lambda * dtd1(r0 - 1, N), 0.0, lambda};
    const M2 CR{lambda, 0.0, c1e, lambda}, CLn{lambda, c1n, 0.0, lambda};
    // coupling of the next block's last two rows to the separator after it
    const int en = e + 2 + base + (t + 1 < extra ? 1 : 0);
    const M2 CRn{lambda, 0.0, lambda * dtd1(en - 1, N), lambda};
    for (int it = 0; it < n_iter; ++it) {
        auto weight = [&](bool hit) { return it == 0 ? 1.0 : (hit ? p : 1.0 - p); };
        // 1. factor the block; corner blocks of its inverse
        M2 br{0.0, 0.0, 0.0, 0.0};
        double2 xl = make_double2(0.0, 0.0);
        if (n > 0) {
            double im1 = 0.0, im2 = 0.0, lm1 = 0.0;       // inverse pivots, L
            double um1 = 0.0, um2 = 0.0, a1 = 0.0, a2 = 0.0, c1 = 0.0, c2 = 0.0;
            M2 tl{0.0, 0.0, 0.0, 0.0};
            double2 xf = make_double2(0.0, 0.0);
            each_row<R>(n, [&](int i) {
                const int g = r0 + i;
                const double w = weight(it > 0 && rows.hit(i));
                // L2 d_{i-2} = lambda, L1 d_{i-1} = b
                const double b = i >= 1 ? lambda * dtd1(g - 1, N) - (i >= 2 ? lambda * lm1 : 0.0)
                                        : 0.0;
                const double L2 = i >= 2 ? lambda * im2 : 0.0, L1 = b * im1;
                const double d = lambda * dtd0(g, N) + w - L2 * lambda - L1 * b;
                const double id = recip(d);
                const double u = w * rows.y(i) - L1 * um1 - L2 * um2;
                // columns 0 and 1 of L^{-1}
                const double ca = (i == 0 ? 1.0 : 0.0) - L1 * a1 - L2 * a2;
                const double cb = (i == 1 ? 1.0 : 0.0) - L1 * c1 - L2 * c2;
                rows.di(i) = id;
                rows.l(i) = L1;
                const double ai = ca * id, bi = cb * id;
                tl.a += ca * ai;
                tl.b += ca * bi;
                tl.d += cb * bi;
                xf.x += ai * u;
                xf.y += bi * u;
                im2 = im1; im1 = id; lm1 = L1;
                um2 = um1; um1 = u;
                a2 = a1; a1 = ca;
                c2 = c1; c1 = cb;
            });
            tl.c = tl.b;
            // columns n-2 and n-1 of L^{-1} are (1, -L_{n-1,n-2}) and (0, 1)
            // on the last two rows and 0 above them
            const double s = -lm1 * im1;
            low_s[t] = BlockLow{tl, M2{a2 * im2 + a1 * s, a1 * im1, c2 * im2 + c1 * s, c1 * im1},
                                xf};
            br = M2{im2 - lm1 * s, s, s, im1};
            xl = make_double2(um2 * im2 + um1 * s, um1 * im1);
        }
        __syncthreads();
        // 2. Schur complement on the separators (separator t lies between
        //    blocks t and t + 1), solved by parallel cyclic reduction
        M2 D{1.0, 0.0, 0.0, 1.0}, up{0.0, 0.0, 0.0, 0.0};
        double2 v = make_double2(0.0, 0.0);
        if (sep) {
            const BlockLow nx = low_s[t + 1];
            const double w0 = weight(hs0), w1 = weight(hs1), c1s = lambda * dtd1(e, N);
            D = sub(sub(M2{lambda * dtd0(e, N) + w0, c1s, c1s, lambda * dtd0(e + 1, N) + w1},
                        mul(tr(CR), mul(br, CR))),
                    mul(tr(CLn), mul(nx.tl, CLn)));
            D.b = D.c = 0.5 * (D.b + D.c);
            v = subv(subv(make_double2(w0 * ys0, w1 * ys1), mulv(tr(CR), xl)),
                     mulv(tr(CLn), nx.xf));
            if (t + 1 < M) up = neg(mul(tr(CLn), mul(nx.trr, CRn)));
        }
        int buf = 0;
        for (int s = 1; s < M; s *= 2, buf ^= 1) {
            if (sep) sep_s[buf][t] = SepRow{inv_sym(D), up, v};
            __syncthreads();
            if (sep) {
                if (t >= s) {
                    const SepRow q = sep_s[buf][t - s];
                    const M2 G = mul(tr(q.up), q.di);
                    D = sub(D, mul(G, q.up));
                    v = subv(v, mulv(G, q.y));
                }
                if (t + s < M) {
                    const SepRow q = sep_s[buf][t + s];
                    const M2 H = mul(up, q.di);
                    D = sub(D, mul(H, tr(up)));
                    v = subv(v, mulv(H, q.y));
                    up = neg(mul(H, q.up));
                }
                D.b = D.c = 0.5 * (D.b + D.c);
            }
        }
        double2 zs = make_double2(0.0, 0.0);
        if (sep) zs_s[t] = zs = mulv(inv_sym(D), v);
        __syncthreads();
        // 3. the block with its separators' values on the right-hand side
        const bool last = it + 1 == n_iter;
        if (n > 0) {
            double2 fl = make_double2(0.0, 0.0), fr = make_double2(0.0, 0.0);
            if (t > 0) fl = mulv(CLt, zs_s[t - 1]);
            if (sep) fr = mulv(CR, zs);
            double um1 = 0.0, um2 = 0.0, im1 = 0.0, im2 = 0.0;
            each_row<R>(n, [&](int i) {
                double r = weight(it > 0 && rows.hit(i)) * rows.y(i);
                if (i == 0) r -= fl.x;
                if (i == 1) r -= fl.y;
                if (i == n - 2) r -= fr.x;
                if (i == n - 1) r -= fr.y;
                const double u = r - rows.l(i) * um1 - (i >= 2 ? lambda * im2 : 0.0) * um2;
                im2 = im1; im1 = rows.di(i);
                rows.u(i) = u;
                um2 = um1; um1 = u;
            });
            double zp1 = 0.0, zp2 = 0.0, lp1 = 0.0;
            each_row_down<R>(n, [&](int i) {
                const double zi = rows.di(i) * (rows.u(i) - (i + 2 < n ? lambda * zp2 : 0.0)) -
                                  (i + 1 < n ? lp1 * zp1 : 0.0);
                lp1 = rows.l(i);
                zp2 = zp1; zp1 = zi;
                rows.set_z(i, zi);
                if (last) zb[r0 + i] = zi;
            });
        }
        hs0 = ys0 > zs.x;
        hs1 = ys1 > zs.y;
        if (last && sep) {
            zb[e] = zs.x;
            zb[e + 1] = zs.y;
        }
    }
}

}  // namespace

}  // namespace xrdvi

using namespace xrdvi;

extern "C" int xrdvi_background(xrdvi_ctx *ctx, int32_t B, int32_t N,
                                const double *y, double lambda, double p,
                                int32_t n_iter, double *bg_out,
                                void *scratch, void *stream) {
    try {
        if (!ctx || !y || !bg_out || !scratch) {
            set_error("background: NULL argument");
            return XRDVI_EINVAL;
        }
        if (B < 1 || N < 1 || n_iter < 1) {
            set_error("background: B, N and n_iter must be >= 1");
            return XRDVI_EINVAL;
        }
        if (!(lambda >= 0.0) || !std::isfinite(lambda) || !(p > 0.0 && p < 0.5)) {
            set_error("background: lambda must be >= 0 and p in (0, 0.5)");
            return XRDVI_EINVAL;
        }
        double *sc = static_cast<double *>(scratch);
        hipStream_t s = static_cast<hipStream_t>(stream);
        // A wave where that has as many threads as the spectrum has blocks (of 8
        // or 9 rows from 48 points on): more spectra then fit a CU (4096 of 100
        // points 140 us, with 256 threads 1053, as one wave with serial separators
        // 668).
        // Rows in registers while blocks are short enough for them.  512 threads
        // have half the registers each: they hold fewer rows, or read the counts
        // again (15 reweightings: 8000 points 187 us with 18 rows and 277 without
        // the counts, 12 000 points 351 us without the counts and 384 with the rows
        // in memory; there 30 000 points take 877, and with each block's rows one
        // after another, which 512 threads cannot keep in a cache, 2700, and 256
        // such spectra more than 64 threads took).
        const auto fits = [N](int threads, int r) { return N <= threads * (r + 2) - 2; };
        constexpr int R1 = 24, R2 = 18;
        const int blocks = (N + 2) / (kMinRows + 2);
        if (blocks <= 64 && blocks >= 5)
            k_asls<64, 10, true><<<B, 64, 0, s>>>(N, y, sc, bg_out, lambda, p, n_iter);
        else if (blocks < 5)
            k_asls<64, R2, true><<<B, 64, 0, s>>>(N, y, sc, bg_out, lambda, p, n_iter);
        else if (fits(256, R1))
            k_asls<256, R1, true><<<B, 256, 0, s>>>(N, y, sc, bg_out, lambda, p, n_iter);
        else if (fits(512, R2))
            k_asls<512, R2, true><<<B, 512, 0, s>>>(N, y, sc, bg_out, lambda, p, n_iter);
        else if (fits(512, R1))
            k_asls<512, R1, false><<<B, 512, 0, s>>>(N, y, sc, bg_out, lambda, p, n_iter);
        else
            k_asls<512, 0, false><<<B, 512, 0, s>>>(N, y, sc, bg_out, lambda, p, n_iter);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            set_error(std::string("background: ") + hipGetErrorString(e));
            return XRDVI_EDEVICE;
        }
        return XRDVI_OK;
    } catch (...) {
        set_error("background: unexpected internal exception");
        return XRDVI_EDEVICE;
    }
}
