"""Strong purely Gaussian peaks on a background of 1e-6 counts, 1e12 times
below them: the profile in the peaks' tails is the Gaussian's value down to
2^-64 of its height, so a sum that ends nearer shows.  Profile against the
FP64 oracle: 1e-5, as for the Gaussian near its centre."""
import numpy as np
import pytest

import oracle
from paper_2501_09308_amd import workloads as W
from paper_2501_09308_amd import xrdvi as X

from gpu_common import context, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sec,asym", [(False, False), (False, True), (True, False)])
@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("cutoff,S", [(0.0, 2), (0.0, 120), (0.0, 300), (8.0, 3)])
def test_gaussian_tails(cutoff, S, merged, sec, asym):
    N, K = 1000, 3
    print(f"\ngaussian tails: c={cutoff} S={S} merged={merged} sec={sec} asym={asym}", flush=True)
    rng = np.random.default_rng(5)
    x = 40.0 + 0.02 * np.arange(N)
    if merged:
        x[600:] = x[599] + 0.01 * np.arange(1, N - 599)
    off = (2 * np.arange(K + 1)).astype(np.int32)
    pos = np.sort(rng.uniform(x[0], x[-1], 2 * K))
    prob = W.Problem(x=x, bg=np.full(N, 1e-6), peak_off=off, peak_pos=pos, peak_int=np.ones(2 * K),
                     cutoff=cutoff, true_idx=np.zeros(0, int), phi_true=np.zeros((4, K)))
    phi = np.zeros((S, 5 if asym else 4, K))
    phi[:, 0] = 1e5 * rng.uniform(0.5, 1.5, (S, K))
    phi[:, 1] = rng.uniform(-0.05, 0.05, (S, K))
    phi[:, 2] = rng.uniform(0.08, 0.12, (S, K))
    if asym:
        phi[:, 4] = rng.uniform(0.8, 1.25, (S, K))
    pro = oracle.profile_sec if sec else oracle.profile_asym if asym else oracle.profile
    ref = pro(x, prob.bg, off, pos, prob.peak_int, cutoff, phi)
    P = X.Problem.from_workload(context(), prob, np.ones(N), cutoff=cutoff, asymmetric=asym,
                                width_law="sec" if sec else 0)
    f = X.xrdvi_profile(context(), P, dev(phi)).cpu().numpy()
    # (the exponent's FP32 rounding is a relative error of 2^-24 q2^2 ln 2, and
    # of a few times that from q2's: 64 x 6e-8 x 4 = 1.5e-5 at the last value
    # that the background does not cover, 2^-64)
    tol = 1e-5 + 2.0 ** -24 * 4.0 * np.log2(np.maximum(ref.max() / ref, 1.0))
    assert np.all(np.abs(f - ref) / ref <= tol)
