"""The dense path's tiles, leaves and nodes against the FP64 oracle at the
sizes where they change: grids of one point, around a leaf (64), a two-leaf
tile (128), a four-leaf tile (256) and the reference block; sample counts on
both sides of each rule of the block cut (one sample per block, four samples
with two or four leaves) and not multiples of four; phases beyond the near
table in LDS (256) and beyond the kept far sums; peaks much wider than a
tile; both width laws, symmetric and asymmetric.  Bars: profile 1e-5, ELBO
and log-likelihoods 1e-6, gradient 1e-4 (the interpolation's error, at most
4.3e-7 of a far peak's term, is far below them)."""
import numpy as np
import pytest

import oracle
from paper_2501_09308_amd import workloads as W
from paper_2501_09308_amd import xrdvi as X

from gpu_common import context, dev, rel_l2

pytestmark = pytest.mark.gpu

# N, S, K, peaks per phase, widest FWHM, asymmetric, sec law
CASES = [
    (1, 3, 4, 6, 0.2, False, False),
    (2, 5, 3, 9, 0.2, True, False),
    (63, 1, 5, 12, 0.2, False, False),
    (65, 4, 5, 12, 0.2, False, True),
    (129, 2, 7, 20, 0.2, True, True),
    (300, 1, 5, 25, 0.2, False, False),
    (129, 200, 3, 8, 0.2, False, False),      # four samples, two leaves
    (257, 131, 4, 10, 0.2, True, False),
    (513, 96, 5, 12, 0.2, False, True),
    (257, 402, 3, 8, 0.2, False, False),      # four leaves, last one of one point
    (1000, 133, 4, 14, 0.2, False, False),
    (900, 150, 3, 10, 0.2, True, False),
    (700, 130, 3, 10, 0.2, False, True),
    (640, 130, 3, 10, 0.2, True, True),
    (400, 6, 259, 3, 0.2, False, False),      # phases beyond the LDS tables
    (700, 130, 130, 2, 0.2, True, False),
    (600, 130, 300, 2, 0.2, False, False),
    (800, 130, 4, 12, 3.0, False, False),     # peaks wider than a tile
    (800, 6, 4, 12, 3.0, True, True),
    (1300, 200, 3, 8, 0.2, False, False),     # the last span cut in two tiles
    (1290, 200, 3, 8, 0.2, True, False),      # ... of which one has points
    (2300, 132, 3, 8, 0.2, False, True),      # two spans
    (2177, 130, 3, 8, 0.2, True, True),
]


@pytest.mark.parametrize("N,S,K,M,wide,asym,sec", CASES)
def test_dense_cut_matches_oracle(N, S, K, M, wide, asym, sec):
    seed = N + 7 * S + 13 * K
    prob = W.make_problem(dict(x0=20.0, step=0.02, N=max(N, 2), K=K, M_range=(1, M), n_true=2,
                               cutoff=0.0, fwhm=(0.05, 0.2)), seed)
    # peaks also outside the scan
    rng = np.random.default_rng(seed)
    prob.peak_pos = rng.uniform(prob.x[0] - 6.0, prob.x[-1] + 6.0, prob.total_peaks)
    if N == 1:
        prob.x, prob.bg = prob.x[:1], prob.bg[:1]
    D = 5 if asym else 4
    pro, el = ((oracle.profile_sec, oracle.elbo_sec) if sec else
               (oracle.profile_asym, oracle.elbo_asym) if asym else
               (oracle.profile, oracle.elbo))
    phi = W.random_phi(K, S, seed + 2, w_range=(0.03, wide))
    if asym:
        phi = np.concatenate([phi, W.random_alpha(K, S, seed + 3)[:, None, :]], axis=1)
    ref = pro(prob.x, prob.bg, prob.peak_off, prob.peak_pos, prob.peak_int, 0.0, phi)
    y = W.poisson_counts(np.maximum(ref[0], prob.bg + 1.0), seed + 1)
    y[0] = max(y[0], prob.bg[0] + 2.0)
    print(f"\ndense nodes: N={N} S={S} K={K} T={prob.total_peaks} asym={asym} sec={sec}", flush=True)
    ctx = context()
    P = X.Problem.from_workload(ctx, prob, y, cutoff=0.0, asymmetric=asym,
                                width_law="sec" if sec else 0)
    f = X.xrdvi_profile(ctx, P, dev(phi)).cpu().numpy()
    assert np.max(np.abs(f - ref) / ref) <= 1e-5
    loc, ls = W.random_params(K, seed + 4, float((y - prob.bg).max()), D=D)
    if wide > 1.0:
        loc[2] += np.log(10.0)          # widths near one degree
    eps = W.eps_draw(S, K, seed + 5, D=D)
    tape = X.Tape(ctx, P, S)
    e, ll = X.xrdvi_elbo_fwd(ctx, P, tape, dev(loc), dev(ls), eps=dev(eps))
    gl, gs = X.xrdvi_elbo_bwd(ctx, tape)
    re, rll, rgl, rgs = el(prob, y, loc, ls, eps)
    assert abs(e.item() - re) <= 1e-6 * abs(re)
    np.testing.assert_allclose(ll.cpu().numpy(), rll, rtol=1e-6)
    g = np.concatenate([gl.cpu().numpy().ravel(), gs.cpu().numpy().ravel()])
    assert rel_l2(g, np.concatenate([rgl.ravel(), rgs.ravel()])) <= 1e-4


@pytest.mark.parametrize("N,S", [(700, 6), (900, 60), (700, 130), (1300, 200)])
def test_each_cut_gives_the_same_bits_served_and_alone(N, S):
    """One dense analysis per kind of block, served together with the others'
    kinds, equals its one-at-a-time run bit for bit."""
    prob = W.make_problem("tiny", seed=N + S, N=N, K=5, M=9)
    fstar = oracle.profile(prob.x, prob.bg, prob.peak_off, prob.peak_pos, prob.peak_int, 0.0,
                           prob.phi_true)[0]
    y = W.poisson_counts(fstar, N + S + 1)
    other = W.make_problem("tiny", seed=5, N=1200, K=4, M=7)
    srv = X.Server(max_slots=4, arena_bytes=1 << 28)
    mine = srv.submit(prob, y, S, 4, 77)
    mix = [srv.submit(other, np.full(1200, 70.0), s, 5, 9) for s in (2, 64, 140)]
    out = None
    for t in [mine] + mix:
        while True:
            rc, _, res = srv.poll(t)
            if rc != X.XRDVI_PENDING:
                break
        assert rc == X.XRDVI_OK
        out = res if t == mine else out
    srv.close()
    ref = X.xrdvi_plain_run(context(), prob, y, S, 4, 77)
    for k in ("loc", "logscale", "trace"):
        assert np.array_equal(out[k], ref[k]), k
