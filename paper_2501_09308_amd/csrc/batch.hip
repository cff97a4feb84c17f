// Batched optimisation step over every resident analysis of the server.
//
// Persistent kernels with fixed grids: each reads the slot table and the
// per-kernel work prefix from device memory, so one captured graph serves
// any membership.  Unit u of a kernel belongs to resident slot i when
// pre[i] <= u < pre[i + 1]; units of analyses that have run all their steps
// do nothing.  The per-unit work is the same device code as the
// single-analysis kernels, and the noise of step n of an analysis is keyed
// by (its seed, n), so an analysis computes the same result alone or in
// any mix.
#include <algorithm>
#include <type_traits>

#include "batch.h"
#include "xrdvi_steps.h"

namespace xrdvi {

namespace {

// Stages the prefix of kernel `kind` and the slot ids in LDS.
struct PrefixSmem {
    int pre[kMaxSlots + 1];
    int slot[kMaxSlots];
    int n;
};

__device__ void load_prefix(const SchedDev *sch, int kind, PrefixSmem &ps) {
    const int n = sch->n;
    for (int i = threadIdx.x; i <= n; i += blockDim.x) ps.pre[i] = sch->pre[kind][i];
    for (int i = threadIdx.x; i < n; i += blockDim.x) ps.slot[i] = sch->slot[i];
    if (threadIdx.x == 0) ps.n = n;
    __syncthreads();
}

__device__ __forceinline__ int uniform(int v) {
    return __builtin_amdgcn_readfirstlane(v);
}

// Resident index i with pre[i] <= u < pre[i + 1] (u is block-uniform, so
// the result is wave-uniform).
__device__ int find_slot(const PrefixSmem &ps, int u) {
    int lo = 0, hi = ps.n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (ps.pre[mid] <= u) lo = mid; else hi = mid;
    }
    return uniform(lo);
}

// Slot table entry of resident index i.  The table does not change while a
// kernel runs, and the index is uniform, so the copy is made of scalar loads
// and the problem and step descriptors stay in scalar registers, as the
// arguments of the single-analysis kernels do.
__device__ __forceinline__ const SlotDev &slot_entry(const SlotDev *tab,
                                                     const PrefixSmem &ps,
                                                     int i) {
    return *(const SlotDev *)(as_const(tab) + uniform(ps.slot[i]));
}

// Unit index of u inside resident index i.
__device__ __forceinline__ int local_unit(const PrefixSmem &ps, int i, int u) {
    return uniform(u - ps.pre[i]);
}

// The units of one kind without the LDS copy, for kernels of many blocks with
// few units each: scalar loads of the prefix, a search for the block's first
// unit, which goes on from there for the next.
struct UnitScan {
    cptr<int> pre, slot;
    int n, total, i = 0;
    __device__ UnitScan(const SchedDev *sch, int kind)
        : pre(as_const(sch->pre[kind])), slot(as_const(sch->slot)),
          n(as_const(&sch->n)[0]), total(pre[n]) {}
    // Resident index of unit u (not below the previous one's).
    __device__ __forceinline__ int at(int u) {
        if (pre[i + 1] <= u) {
            int hi = n;
            ++i;
            while (hi - i > 1) {
                const int mid = (i + hi) >> 1;
                if (pre[mid] <= u) i = mid; else hi = mid;
            }
        }
        return i;
    }
};

__device__ inline bool running(const SlotDev &d) {
    return uniform(*d.step) < d.steps;
}

}  // namespace

__global__ __launch_bounds__(256) void kb_sample(const SlotDev *tab,
                                                 const SchedDev *sch) {
    __shared__ PrefixSmem ps;
    __shared__ SampleSmem sm;
    load_prefix(sch, kSample, ps);
    const int total = uniform(ps.pre[ps.n]);
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int i = find_slot(ps, u);
        const SlotDev &d = slot_entry(tab, ps, i);
        if (!running(d)) continue;
        const int local = local_unit(ps, i, u);
        const int nkb = (d.P.K + kWave - 1) / kWave;
        if (local / nkb >= d.st.S) continue;
        sample_block(d.P, d.st, d.loc, d.logscale, nullptr, d.seed,
                     (uint64_t)*d.step, local / nkb, local % nkb, nkb, sm);
        __syncthreads();
    }
}

// The window step.  With a constant width (windowed analyses) an
// analysis's first ceil(K / 64) units find its phases' extremes over the
// samples instead, 64 phases each (see batch_units).
template <bool SEC>
__global__ __launch_bounds__(256) void kb_windows(const SlotDev *tab,
                                                  const SchedDev *sch) {
    __shared__ PrefixSmem ps;
    __shared__ typename std::conditional<SEC, char, CandExtSmem>::type sm;
    load_prefix(sch, SEC ? kWindowsSec : kWindows, ps);
    const int total = uniform(ps.pre[ps.n]);
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int i = find_slot(ps, u);
        const SlotDev &d = slot_entry(tab, ps, i);
        if (!running(d)) continue;
        int local = local_unit(ps, i, u);
        if constexpr (!SEC) {
            const int next = (d.P.K + kWave - 1) / kWave;
            if (local < next) {
                if (d.st.cab) cand_ext_block(d.P, d.st, d.st.phi, local * kWave, sm);
                __syncthreads();   // the extremes' LDS is reused by the next unit
                continue;
            }
            local -= next;
        }
        windows_elem<SEC>(d.P, d.st.S, d.st.phi, d.P.cutoff > 0.0 ? d.st.lo : nullptr,
                          d.st.hi, nullptr, (size_t)local * 256, d.st.psec);
    }
}

__global__ __launch_bounds__(kCandThreads) void kb_cand(const SlotDev *tab,
                                                        const SchedDev *sch) {
    __shared__ PrefixSmem ps;
    load_prefix(sch, kCand, ps);
    const int total = uniform(ps.pre[ps.n]);
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int i = find_slot(ps, u);
        const SlotDev &d = slot_entry(tab, ps, i);
        if (!running(d) || !d.st.cab) continue;
        const int local = local_unit(ps, i, u);
        const int nkb = (d.P.K + kCandThreads - 1) / kCandThreads;
        const int t = local / nkb, k = (local % nkb) * kCandThreads + threadIdx.x;
        if (t < d.P.ntiles && k < d.P.K) cand_elem(d.P, d.st, t, k);
    }
}

// Held to the blocks per CU the LDS allows, as the single-analysis kernel (a
// few values are spilled once per block and reloaded once per unit, outside
// the record loops).  With the prefix in LDS six fit, and every block loaded
// it: eight analyses (N 2000-12000, K 20-300, S 32) 141 us a step, now 136;
// the adjoint 143, now 138.
template <bool ASYM, bool SEC>
__global__ __launch_bounds__(kBlock, ASYM || SEC ? 6 : 7) void kb_win(const SlotDev *tab, const SchedDev *sch) {
    __shared__ WinSmem<ASYM> sm;
    UnitScan us(sch, fused_kind(true, ASYM, SEC));
    for (int u = blockIdx.x; u < us.total; u += gridDim.x) {
        const int i = us.at(u);
        const SlotDev &d = *(const SlotDev *)(as_const(tab) + us.slot[i]);
        if (!running(d)) continue;
        const int local = u - us.pre[i];
        int t = local % d.P.ntiles, s = local / d.P.ntiles;
        if (d.st.S % kXcds == 0) {
            // a block runs on XCD u mod 8, and u - local is the same for all
            // of an analysis's units: the units with one value of local mod 8
            // share an XCD, which takes one eighth of the samples of every
            // tile (its L2 keeps those samples' window arrays)
            const int G = d.st.S / kXcds, q = local / kXcds;
            t = q / G;
            s = (local % kXcds) * G + q % G;
        }
        if (s >= d.st.S) continue;
        // records in grid steps on a uniform grid (constant width only)
        if (!SEC && uses_grid_steps(d.P))
            win_tile<ASYM, SEC, !SEC>(d.P, d.st, t, s, nullptr, sm);
        else
            win_tile<ASYM, SEC, false>(d.P, d.st, t, s, nullptr, sm);
        __syncthreads();
    }
}

// Dense fused forward + adjoint, units (tile, sample group) with the groups
// fastest (a tile's samples run at the same time and share its peaks).  SG: the
// units of analyses with that many samples per block, the others pass by; with
// one, two blocks share a CU as in the single-analysis kernel.
template <bool ASYM, bool SEC, int SG>
union DenseBatchSmem {
    DenseSmem<kDenseWaves, SG, 2, ASYM, SEC> two;
    DirectSmem<kDenseWaves, SG, 2, ASYM> dtwo;
};
template <bool ASYM, bool SEC>
union DenseBatchSmem<ASYM, SEC, 4> {
    DenseSmem<kDenseWaves, 4, 4, ASYM, SEC> wide;
    DenseSmem<kDenseWaves, 4, 2, ASYM, SEC> two;
    DirectSmem<kDenseWaves, 4, 4, ASYM> dwide;
    DirectSmem<kDenseWaves, 4, 2, ASYM> dtwo;
};
template <bool ASYM, bool SEC, int SG>
__global__ __launch_bounds__(kDenseWaves * kWave, SG == 1 ? 8 : 4) void kb_dense(
    const SlotDev *tab, const SchedDev *sch) {
    __shared__ PrefixSmem ps;
    __shared__ DenseBatchSmem<ASYM, SEC, SG> sm;
    load_prefix(sch, fused_kind(false, ASYM, SEC), ps);
    const int total = uniform(ps.pre[ps.n]);
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int i = find_slot(ps, u);
        const SlotDev &d = slot_entry(tab, ps, i);
        const DenseCut cut = dense_cut(d.P.N, d.st.S);
        if (cut.group != SG || !running(d)) continue;
        const int local = local_unit(ps, i, u);
        const int ng = cut.groups(d.st.S), t = local / ng, grp = local % ng;
        if (t >= d.st.nt) continue;
        const int wide = cut.wide(d.P.N);   // tiles of cut.leaves, then of two
        const bool is_wide = SG == 4 && cut.leaves == 4 && t < wide;
        const int tw = SG == 4 && cut.leaves == 4 ? t + wide : t;   // ... as one of two
        const auto tile = [&](auto cut_tag) {
            constexpr bool CUT = decltype(cut_tag)::value;
            if constexpr (SG == 4) {
                if (is_wide) {
                    dense_tile<true, ASYM, SEC, kDenseWaves, 4, 4, CUT>(d.P, d.st, t, t, grp,
                                                                        nullptr, sm.wide);
                    return;
                }
            }
            dense_tile<true, ASYM, SEC, kDenseWaves, SG, 2, CUT>(d.P, d.st, tw, t, grp, nullptr,
                                                                 sm.two);
        };
        if (direct_peaks<SG, ASYM>(d.P.K, d.P.T)) {
            if constexpr (SG == 4) {
                if (is_wide)
                    dense_direct<true, ASYM, SEC, kDenseWaves, 4, 4>(d.P, d.st, t, t, grp,
                                                                     nullptr, sm.dwide);
            }
            if (!is_wide)
                dense_direct<true, ASYM, SEC, kDenseWaves, SG, 2>(d.P, d.st, tw, t, grp, nullptr,
                                                                  sm.dtwo);
        } else if (cut_phases(d.P.K)) {
            tile(std::true_type{});
        } else {
            tile(std::false_type{});
        }
        __syncthreads();
    }
}

template <bool ASYM, bool SEC>
__global__ __launch_bounds__(kBlock, ASYM ? (SEC ? 5 : 6) : (SEC ? 7 : 8)) void kb_adjoint(const SlotDev *tab,
                                                     const SchedDev *sch) {
    __shared__ double red[kWaves][12];
    __shared__ ElboSmem<kBlock> el;
    UnitScan us(sch, adjoint_kind(ASYM, SEC));
    for (int u = blockIdx.x; u < us.total; u += gridDim.x) {
        const int i = us.at(u);
        const SlotDev &d = *(const SlotDev *)(as_const(tab) + us.slot[i]);
        if (!running(d)) continue;
        const int local = u - us.pre[i];
        if (d.P.cutoff == 0.0) continue;
        if (local / d.P.K >= d.st.S) {        // the ELBO
            const double e = elbo_block<kBlock>(d.P, d.st, d.logscale, nullptr, el);
            if (threadIdx.x == 0) d.trace[*d.step] = e;
            __syncthreads();
            continue;
        }
        if (d.P.few)
            adjoint_phase<ASYM, SEC, kWave>(d.P, d.st, local / d.P.K, local % d.P.K, red);
        else
            adjoint_phase<ASYM, SEC, kAdjLanes>(d.P, d.st, local / d.P.K, local % d.P.K, red);
        __syncthreads();
    }
}

__global__ __launch_bounds__(1024) void kb_elbo(const SlotDev *tab,
                                                const SchedDev *sch) {
    __shared__ PrefixSmem ps;
    __shared__ ElboSmem<1024> sm;
    load_prefix(sch, kElbo, ps);
    const int total = uniform(ps.pre[ps.n]);
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int i = find_slot(ps, u);
        const SlotDev &d = slot_entry(tab, ps, i);
        if (!running(d)) continue;
        const double e = elbo_block<1024>(d.P, d.st, d.logscale, nullptr, sm);
        if (threadIdx.x == 0) d.trace[*d.step] = e;
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void kb_grad_adam(const SlotDev *tab,
                                                    const SchedDev *sch) {
    __shared__ PrefixSmem ps;
    __shared__ GradSmem sm;
    load_prefix(sch, kGrad, ps);
    const int total = uniform(ps.pre[ps.n]);
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int i = find_slot(ps, u);
        const SlotDev &d = slot_entry(tab, ps, i);
        if (!running(d)) continue;
        AdamArgs a;
        a.m1_loc = d.m1_loc; a.m2_loc = d.m2_loc;
        a.m1_ls = d.m1_ls; a.m2_ls = d.m2_ls;
        a.t = *d.step + 1;
        a.lr = d.lr; a.b1 = 0.9; a.b2 = 0.999; a.eps = 1e-8;
        if (d.P.cutoff > 0.0) {
            // windowed: one phase per wave
            const int k = local_unit(ps, i, u) * kWaves + (int)(threadIdx.x / kWave);
            if (k < d.P.K)
                grad_wave(d.P, d.st, k, 1.0, nullptr, nullptr, nullptr, d.loc,
                          d.logscale, &a);
        } else {
            const int k = local_unit(ps, i, u);
            if (k >= d.P.K) continue;
            grad_block(d.P, d.st, k, 1.0, nullptr, nullptr, nullptr,
                       d.loc, d.logscale, &a, sm);
        }
        __syncthreads();
    }
}

// Last kernel of a step: every running analysis moves to its next step.
__global__ void kb_advance(const SlotDev *tab, const SchedDev *sch) {
    const int n = sch->n;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += gridDim.x * blockDim.x) {
        const SlotDev &d = tab[sch->slot[i]];
        if (*d.step < d.steps) *d.step += 1;
    }
}

// An analysis's table entry, step counter and trace in one launch; the entry
// travels as a kernel argument.
__global__ __launch_bounds__(256) void kb_enter(SlotDev d, SlotDev *entry) {
    const int g = blockIdx.x * 256 + threadIdx.x;
    for (int n = g; n < d.steps; n += gridDim.x * 256) d.trace[n] = 0.0;
    if (g == 0) {
        *entry = d;
        *d.step = 0;
    }
}

hipError_t launch_enter_slot(const SlotDev &d, SlotDev *entry, hipStream_t s) {
    kb_enter<<<std::min((d.steps + 255) / 256, 256), 256, 0, s>>>(d, entry);
    return hipGetLastError();
}

template <bool ASYM, bool SEC>
static void launch_dense(const SlotDev *tab, const SchedDev *sch, hipStream_t s,
                         unsigned classes) {
    if (classes & kDenseFour)
        kb_dense<ASYM, SEC, 4><<<kGridDense, kDenseWaves * kWave, 0, s>>>(tab, sch);
    if (classes & kDenseOne)
        kb_dense<ASYM, SEC, 1><<<2 * kGridDense, kDenseWaves * kWave, 0, s>>>(tab, sch);
}

hipError_t launch_batch_step(const SlotDev *tab, const SchedDev *sch,
                             hipStream_t s, unsigned classes) {
    // whether a resident class satisfies the windowed / sec-law test
    const auto any = [classes](int want_win, int want_sec) {
        for (int c = 0; c < 8; ++c)
            if ((classes >> c & 1u) && (want_win < 0 || (c & 1) == want_win) &&
                (want_sec < 0 || (c >> 2 & 1) == want_sec))
                return true;
        return false;
    };
    const auto has = [classes](bool win, bool asym, bool sec) {
        return (classes >> ((win ? 1 : 0) | (asym ? 2 : 0) | (sec ? 4 : 0)) & 1u) != 0;
    };
    kb_sample<<<kGridSmall, 256, 0, s>>>(tab, sch);
    if (any(1, 0)) kb_windows<false><<<kGridLarge, 256, 0, s>>>(tab, sch);
    if (any(-1, 1)) kb_windows<true><<<kGridLarge, 256, 0, s>>>(tab, sch);
    if (any(1, 0)) kb_cand<<<kGridLarge, kCandThreads, 0, s>>>(tab, sch);
    if (has(true, false, false)) kb_win<false, false><<<kGridWin, kBlock, 0, s>>>(tab, sch);
    if (has(false, false, false)) launch_dense<false, false>(tab, sch, s, classes);
    if (has(true, true, false)) kb_win<true, false><<<kGridWin, kBlock, 0, s>>>(tab, sch);
    if (has(false, true, false)) launch_dense<true, false>(tab, sch, s, classes);
    if (has(true, false, true)) kb_win<false, true><<<kGridWin, kBlock, 0, s>>>(tab, sch);
    if (has(false, false, true)) launch_dense<false, true>(tab, sch, s, classes);
    if (has(true, true, true)) kb_win<true, true><<<kGridWin, kBlock, 0, s>>>(tab, sch);
    if (has(false, true, true)) launch_dense<true, true>(tab, sch, s, classes);
    if (has(true, false, false)) kb_adjoint<false, false><<<kGridAdjoint, kBlock, 0, s>>>(tab, sch);
    if (has(true, true, false)) kb_adjoint<true, false><<<kGridAdjoint, kBlock, 0, s>>>(tab, sch);
    if (has(true, false, true)) kb_adjoint<false, true><<<kGridAdjoint, kBlock, 0, s>>>(tab, sch);
    if (has(true, true, true)) kb_adjoint<true, true><<<kGridAdjoint, kBlock, 0, s>>>(tab, sch);
    if (any(0, -1)) kb_elbo<<<kGridElbo, 1024, 0, s>>>(tab, sch);
    kb_grad_adam<<<kGridLarge, 256, 0, s>>>(tab, sch);
    kb_advance<<<1, 1024, 0, s>>>(tab, sch);
    return hipGetLastError();
}

}  // namespace xrdvi
