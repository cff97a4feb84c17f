"""The windowed forward's peak ranges: windows that end on a tile's first point
for shifts and widths of 900 deg that cancel, where the FP32 bounds' terms round
by more than the peaks' positions.  Profile against the FP64 oracle: 1e-5."""
import numpy as np
import pytest

import oracle
from paper_2501_09308_amd import workloads as W
from paper_2501_09308_amd import xrdvi as X

from gpu_common import context, dev

pytestmark = pytest.mark.gpu


def _problem(x, bg, M, pos, inten, cutoff):
    off = np.concatenate([[0], np.cumsum(M)]).astype(np.int32)
    K = len(M)
    return W.Problem(x=x, bg=np.full(x.size, bg), peak_off=off, peak_pos=pos, peak_int=inten,
                     cutoff=cutoff, true_idx=np.zeros(0, int), phi_true=np.zeros((4, K)))


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
