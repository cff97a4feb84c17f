"""The windowed adjoint of problems of few peaks per phase (at most eight: one
peak at a time on a whole wave) and just beyond, with short and long windows,
uniform and merged grids, every width law; alone against the FP64 oracle
(gradient 1e-4 by latent) and served, the same bits."""
import math

import numpy as np
import pytest

import oracle
from paper_2501_09308_amd import workloads as W
from paper_2501_09308_amd import xrdvi as X

from gpu_common import context, dev, rel_l2

pytestmark = pytest.mark.gpu


def _problem(M, merged, cutoff):
    N, K = 900, len(M)
    rng = np.random.default_rng(sum(M) + K)
    x = 40.0 + 0.02 * np.arange(N)
    if merged:
        x[500:] = x[499] + 0.01 * np.arange(1, N - 499)
    off = np.concatenate([[0], np.cumsum(M)]).astype(np.int32)
    T = int(off[-1])
    return W.Problem(x=x, bg=np.full(N, 20.0), peak_off=off,
                     peak_pos=rng.uniform(x[0] - 1.0, x[-1] + 1.0, T),
                     peak_int=rng.uniform(0.2, 1.0, T), cutoff=cutoff,
                     true_idx=np.zeros(0, int), phi_true=np.zeros((4, K)))


@pytest.mark.parametrize("asym,sec", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("w", [0.05, 0.5])
@pytest.mark.parametrize("M", [(1,), (3, 1, 4), (8, 0, 5, 7), (9, 2), (6, 8)])
def test_few_peaks(M, w, merged, asym, sec):
    S, K, D = 5, len(M), 5 if asym else 4
    print(f"\nfew peaks: M={M} w={w} merged={merged} asym={asym} sec={sec}", flush=True)
    prob = _problem(M, merged, 8.0)
    rng = np.random.default_rng(K)
    loc = np.zeros((D, K))
    loc[0] = math.log(20.0) + 0.3 * rng.standard_normal(K)
    loc[1] = 0.02 * rng.standard_normal(K)
    loc[2] = math.log(w) + 0.2 * rng.standard_normal(K)
    loc[3] = rng.standard_normal(K)
    if asym:
        loc[4] = 0.2 * rng.standard_normal(K)
    ls = np.full((D, K), math.log(0.05))
    eps = rng.standard_normal((S, D, K))
    el = oracle.elbo_sec if sec else oracle.elbo_asym if asym else oracle.elbo
    y = rng.poisson(40.0, prob.N).astype(float)
    ctx = context()
    P = X.Problem.from_workload(ctx, prob, y, cutoff=8.0, asymmetric=asym,
                                width_law="sec" if sec else 0)
    tape = X.Tape(ctx, P, S)
    X.xrdvi_elbo_fwd(ctx, P, tape, dev(loc), dev(ls), eps=dev(eps))
    gl, gs = X.xrdvi_elbo_bwd(ctx, tape)
    _, _, rgl, rgs = el(prob, y, loc, ls, eps)
    for row in range(D):
        assert rel_l2(gl.cpu().numpy()[row], rgl[row]) <= 1e-4, row
        assert rel_l2(gs.cpu().numpy()[row], rgs[row]) <= 1e-4, row


def test_few_peaks_served_beside_many():
    few, many = _problem((3, 1, 8), False, 8.0), _problem((20, 9), False, 8.0)
    y = np.random.default_rng(1).poisson(40.0, few.N).astype(float)
    srv = X.Server(max_slots=4, arena_bytes=1 << 28)
    tickets = [(srv.submit(p, y, 8, 4, 5), p) for p in (few, many)]
    outs = []
    for t, _ in tickets:
        while True:
            rc, _, out = srv.poll(t)
            if rc != X.XRDVI_PENDING:
                break
        assert rc == X.XRDVI_OK
        outs.append(out)
    srv.close()
    for out, (_, p) in zip(outs, tickets):
        ref = X.xrdvi_plain_run(context(), p, y, 8, 4, 5)
        for k in ("loc", "logscale", "trace"):
            assert np.array_equal(out[k], ref[k]), k
