"""The windowed forward's peak ranges: phases with more peaks on a tile than are
counted one by one (16), on both sides of that number and far more than the
staging space holds; and windows that end on a tile's first point for shifts and
widths of 900 deg that cancel, where the FP32 bounds' terms round by more than
the peaks' positions.  Against the FP64 oracle: profile 1e-5, ELBO 1e-6,
gradient 1e-4."""
import math

import numpy as np
import pytest

import oracle
from paper_2501_09308_amd import workloads as W
from paper_2501_09308_amd import xrdvi as X

from gpu_common import context, dev, rel_l2

pytestmark = pytest.mark.gpu


def _problem(x, bg, M, pos, inten, cutoff):
    off = np.concatenate([[0], np.cumsum(M)]).astype(np.int32)
    K = len(M)
    return W.Problem(x=x, bg=np.full(x.size, bg), peak_off=off, peak_pos=pos, peak_int=inten,
                     cutoff=cutoff, true_idx=np.zeros(0, int), phi_true=np.zeros((4, K)))


@pytest.mark.parametrize("asym,sec", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("M,w", [((15, 16, 17, 18, 4, 33), 0.5), ((150, 0, 16, 90, 17), 0.25),
                                 ((400, 300, 500), 0.3), ((64, 20, 40), 4.0)])
def test_many_peaks_on_a_tile(M, w, merged, asym, sec):
    N, S, K, D = 700, 3, len(M), 5 if asym else 4
    print(f"\nmany peaks: M={M} w={w} merged={merged} asym={asym} sec={sec}", flush=True)
    rng = np.random.default_rng(sum(M))
    x = 50.0 + 0.02 * np.arange(N)
    if merged:
        x[400:] = x[399] + 0.01 * np.arange(1, N - 399)
    prob = _problem(x, 20.0, M, rng.uniform(x[0] - 3.0, x[-1] + 3.0, sum(M)),
                    rng.uniform(0.2, 1.0, sum(M)), 8.0)
    loc = np.zeros((D, K))
    loc[0] = math.log(20.0) + 0.3 * rng.standard_normal(K)
    loc[1] = 0.05 * rng.standard_normal(K)
    loc[2] = math.log(w) + 0.2 * rng.standard_normal(K)
    loc[3] = rng.standard_normal(K)
    if asym:
        loc[4] = 0.2 * rng.standard_normal(K)
    ls = np.full((D, K), math.log(0.05))
    eps = rng.standard_normal((S, D, K))
    z = loc + np.exp(ls) * eps
    phi = np.exp(z)
    phi[:, 1] = z[:, 1]
    phi[:, 3] = 1.0 / (1.0 + np.exp(-z[:, 3]))
    pro, el = ((oracle.profile_sec, oracle.elbo_sec) if sec else
               (oracle.profile_asym, oracle.elbo_asym) if asym else
               (oracle.profile, oracle.elbo))
    ref = pro(x, prob.bg, prob.peak_off, prob.peak_pos, prob.peak_int, 8.0, phi)
    y = np.floor(1.5 * ref[0] + 3.0)
    ctx = context()
    P = X.Problem.from_workload(ctx, prob, y, cutoff=8.0, asymmetric=asym,
                                width_law="sec" if sec else 0)
    f = X.xrdvi_profile(ctx, P, dev(phi)).cpu().numpy()
    assert np.max(np.abs(f - ref) / ref) <= 1e-5
    tape = X.Tape(ctx, P, S)
    e, _ = X.xrdvi_elbo_fwd(ctx, P, tape, dev(loc), dev(ls), eps=dev(eps))
    gl, gs = X.xrdvi_elbo_bwd(ctx, tape)
    re, _, rgl, rgs = el(prob, y, loc, ls, eps)
    assert abs(e.item() - re) <= 1e-6 * abs(re)
    g = np.concatenate([gl.cpu().numpy().ravel(), gs.cpu().numpy().ravel()])
    assert rel_l2(g, np.concatenate([rgl.ravel(), rgs.ravel()])) <= 1e-4


@pytest.mark.parametrize("n", [1, 40])
def test_windows_of_large_shifts_end_on_a_tile(n):
    """Peak q (of n at one place) ends its window 1e-8 deg past the first point
    of the third tile: the point has its value, the next one not."""
    N, S = 512, 64
    print(f"\nlarge shifts: n={n}", flush=True)
    x = 60.0 + 0.02 * np.arange(N)
    prob = _problem(x, 1e-3, (n,), np.full(n, x[256] + 1e-8), np.ones(n), 8.0)
    phi = np.zeros((S, 4, 1))
    shift = 900.0 + 0.01317 * np.arange(S)
    phi[:, 0, 0] = 10.0
    phi[:, 1, 0] = -shift
    phi[:, 2, 0] = shift / 8.0
    phi[:, 3, 0] = 1.0
    ref = oracle.profile(x, prob.bg, prob.peak_off, prob.peak_pos, prob.peak_int, 8.0, phi)
    assert np.all(ref[:, 256] > 1.1 * ref[:, 257])
    P = X.Problem.from_workload(context(), prob, np.ones(N), cutoff=8.0)
    f = X.xrdvi_profile(context(), P, dev(phi)).cpu().numpy()
    assert np.max(np.abs(f - ref) / ref) <= 1e-5
