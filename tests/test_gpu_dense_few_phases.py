"""Dense analyses of few phases, whose peaks several waves share: one to nine
phases (the rule ends at eight), of no peaks, fewer than shares, one, and many,
and so few peaks that every one is taken at every point, in every kind of block,
against the FP64 oracle: profile 1e-5, ELBO 1e-6, each phase's and latent's
gradient 1e-4; and served, the same bits as alone."""
import math

import numpy as np
import pytest

import oracle
from paper_2501_09308_amd import workloads as W
from paper_2501_09308_amd import xrdvi as X

from gpu_common import context, dev, rel_l2

pytestmark = pytest.mark.gpu


def _case(N, S, M, D):
    K = len(M)
    rng = np.random.default_rng(N + S + K)
    x = 30.0 + 0.02 * np.arange(N)
    off = np.concatenate([[0], np.cumsum(M)]).astype(np.int32)
    T = int(off[-1])
    prob = W.Problem(x=x, bg=np.full(N, 5.0), peak_off=off,
                     peak_pos=rng.uniform(x[0] - 3.0, x[-1] + 3.0, T),
                     peak_int=rng.uniform(0.2, 1.0, T), cutoff=0.0,
                     true_idx=np.zeros(0, int), phi_true=np.zeros((4, K)))
    loc = np.zeros((D, K))
    loc[0] = math.log(20.0) + 0.3 * rng.standard_normal(K)
    loc[1] = 0.02 * rng.standard_normal(K)
    loc[2] = math.log(0.1) + 0.2 * rng.standard_normal(K)
    loc[3] = rng.standard_normal(K)
    if D == 5:
        loc[4] = 0.2 * rng.standard_normal(K)
    return prob, loc, np.full((D, K), math.log(0.05)), rng.standard_normal((S, D, K))


@pytest.mark.parametrize("asym,sec", [(False, False), (True, False), (False, True)])
@pytest.mark.parametrize("N,S", [(90, 2), (700, 1), (900, 61), (700, 130), (1300, 200)])
@pytest.mark.parametrize("M", [(150,), (1,), (40, 0), (3, 17, 400), (5, 1, 0, 20, 9),
                               (2, 9, 30, 1, 16, 15, 17, 40), (4, 9, 30, 1, 0, 15, 17, 40, 8),
                               (53,), (54,), (20, 30), (20, 31), 14 * (1,), 17 * (0,) + (2,),
                               (50,), 8 * (1,)])
def test_few_phases(M, N, S, asym, sec):
    print(f"\nfew phases: M={M} N={N} S={S} asym={asym} sec={sec}", flush=True)
    prob, loc, ls, eps = _case(N, S, M, 5 if asym else 4)
    z = loc + np.exp(ls) * eps
    phi = np.exp(z)
    phi[:, 1] = z[:, 1]
    phi[:, 3] = 1.0 / (1.0 + np.exp(-z[:, 3]))
    pro, el = ((oracle.profile_sec, oracle.elbo_sec) if sec else
               (oracle.profile_asym, oracle.elbo_asym) if asym else
               (oracle.profile, oracle.elbo))
    ref = pro(prob.x, prob.bg, prob.peak_off, prob.peak_pos, prob.peak_int, 0.0, phi)
    y = np.floor(1.5 * ref[0] + 3.0)
    ctx = context()
    P = X.Problem.from_workload(ctx, prob, y, cutoff=0.0, asymmetric=asym,
                                width_law="sec" if sec else 0)
    f = X.xrdvi_profile(ctx, P, dev(phi)).cpu().numpy()
    assert np.max(np.abs(f - ref) / ref) <= 1e-5
    tape = X.Tape(ctx, P, S)
    e, _ = X.xrdvi_elbo_fwd(ctx, P, tape, dev(loc), dev(ls), eps=dev(eps))
    gl, gs = X.xrdvi_elbo_bwd(ctx, tape)
    re, _, rgl, rgs = el(prob, y, loc, ls, eps)
    assert abs(e.item() - re) <= 1e-6 * abs(re)
    for k in range(len(M)):
        assert rel_l2(gl.cpu().numpy()[:, k], rgl[:, k]) <= 1e-4, k
        assert rel_l2(gs.cpu().numpy()[:, k], rgs[:, k]) <= 1e-4, k


@pytest.mark.parametrize("M", [(50, 3, 20), (5, 1, 0, 20, 9)])
@pytest.mark.parametrize("N,S", [(700, 6), (900, 60), (1300, 200)])
def test_few_phases_served(N, S, M):
    prob, _, _, _ = _case(N, S, M, 4)
    y = np.random.default_rng(1).poisson(40.0, N).astype(float)
    srv = X.Server(max_slots=2, arena_bytes=1 << 28)
    ticket = srv.submit(prob, y, S, 4, 77)
    while True:
        rc, _, out = srv.poll(ticket)
        if rc != X.XRDVI_PENDING:
            break
    assert rc == X.XRDVI_OK
    srv.close()
    ref = X.xrdvi_plain_run(context(), prob, y, S, 4, 77)
    for k in ("loc", "logscale", "trace"):
        assert np.array_equal(out[k], ref[k]), k
