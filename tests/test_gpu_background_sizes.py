"""The background where one wave takes a spectrum (to 647 points) and where the
rows lie in memory (from 13 311): both sides of each rule, several spectra at
once, each against the oracle's sparse solve of that spectrum.  Bar: two
direct solves agree, normwise, to the condition number (1 + 16 lambda / p) times
the FP64 epsilon, 7e-10 here."""
import numpy as np
import pytest
import torch

from oracle import background as BG
from paper_2501_09308_amd import xrdvi as X

from gpu_common import context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B", [(1, 3), (2, 3), (4, 1), (27, 3), (28, 3), (47, 5), (48, 5),
                                 (57, 2), (333, 300), (647, 4), (648, 4), (13310, 3),
                                 (13311, 3), (15007, 2), (40001, 1)])
def test_background_sizes(N, B):
    lam, p, n_iter = 1e3, 0.01, 5
    print(f"\nbackground: N={N} B={B}", flush=True)
    rng = np.random.default_rng(N)
    x = np.linspace(0.0, 70.0, N)
    f = 60.0 + 150.0 * np.exp(-x / 20.0) + sum(
        800.0 * rng.uniform() / (1.0 + ((x - c) / 0.1) ** 2) for c in rng.uniform(0.0, 70.0, 20))
    y = rng.poisson(f, size=(B, N)).astype(np.float64)
    out = X.xrdvi_background(context(), torch.as_tensor(y, device="cuda"), lam, p,
                             n_iter).cpu().numpy()
    rtol = 2.0 * (1.0 + 16.0 * lam / p) * 2.2e-16
    for b in range(min(B, 8)):
        ref = BG.asls(y[b], lam, p, n_iter) if N > 2 else y[b]
        assert np.max(np.abs(out[b] - ref)) / np.max(np.abs(ref)) <= rtol
    if B > 8:                          # the last spectra alone
        one = X.xrdvi_background(context(), torch.as_tensor(y[-2:].copy(), device="cuda"), lam, p,
                                 n_iter).cpu().numpy()
        assert np.array_equal(one, out[-2:])
