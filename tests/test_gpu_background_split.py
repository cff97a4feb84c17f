"""The background's parallel split against the oracle's sparse solve at the
sizes where the split changes: the fewest rows and blocks, the last size of
each kernel (256 threads with 24 rows each, 512 with 18, 512 with 24) and the
first of the next, and several spectra at once; with no smoothness and with a
stiff penalty.  Bar: two direct solves agree, normwise, to the condition
number (1 + 16 lambda / p) times the FP64 epsilon."""
import numpy as np
import pytest
import torch

from oracle import background as BG
from paper_2501_09308_amd import xrdvi as X

from gpu_common import context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B,lam", [(3, 1, 10.0), (17, 2, 10.0), (18, 2, 10.0), (38, 1, 0.0),
                                     (2558, 1, 1e5), (2559, 5, 1e5), (6654, 1, 1e6),
                                     (6655, 2, 1e6), (10238, 1, 1e7), (10239, 1, 1e7),
                                     (13310, 2, 1e6), (13311, 1, 1e6)])
def test_background_split_matches_oracle(N, B, lam):
    p, n_iter = 0.01, 4
    rng = np.random.default_rng(N)
    x = np.linspace(0.0, 70.0, N)
    f = 60.0 + 150.0 * np.exp(-x / 20.0) + sum(
        800.0 * rng.uniform() / (1.0 + ((x - c) / 0.1) ** 2) for c in rng.uniform(0.0, 70.0, 20))
    y = rng.poisson(f, size=(B, N)).astype(np.float64)
    out = X.xrdvi_background(context(), torch.as_tensor(y, device="cuda"), lam, p,
                             n_iter).cpu().numpy()
    rtol = 2.0 * (1.0 + 16.0 * lam / p) * 2.2e-16
    for b in range(B):
        ref = BG.asls(y[b], lam, p, n_iter)
        err = np.max(np.abs(out[b] - ref)) / np.max(np.abs(ref))
        assert err <= max(rtol, 1e-12), (err, rtol)
