"""Window bounds that fall on, next to and between grid points.

On a uniform grid a bound clearly between two points is counted without a look
at the grid; one near a point, and every bound on other grids, is searched.
Both must give exactly the range of the definition, rho - c w <= x_i <= rho +
c w in FP64, for fewer and for more peaks than a block has threads.
"""
import numpy as np
import pytest
import torch

from paper_2501_09308_amd import xrdvi as X
from gpu_common import context, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 7, 255, 256, 257, 900])
@pytest.mark.parametrize("grid", ["uniform", "jittered", "merged", "one"])
def test_windows_are_the_definition_s(grid, T):
    rng = np.random.default_rng([3, T, len(grid)])
    N, S, c, w = 1201, 5, 8.0, 0.125
    x = 10.0 + 0.0625 * np.arange(N)          # steps and widths exact in FP64
    if grid == "jittered":                     # uniform within the recognised error
        x = x + 3e-11 * rng.uniform(-1, 1, N)
    elif grid == "merged":
        x = np.concatenate([x[:700], x[699] + 0.03125 * np.arange(1, N - 699)])
    elif grid == "one":
        x, N = x[:1], 1
    # centres whose bounds lie on points, within 1e-12 .. 1e-3 of them, between
    # them, and past both ends of the grid
    pos = rng.uniform(x[0] - 2.0, x[-1] + 2.0, T)
    snap = rng.random(T) < 0.7
    pos[snap] = x[rng.integers(0, N, snap.sum())]
    pos += rng.choice([0.0, 1e-12, -1e-12, 6e-11, -6e-11, 1e-7, -1e-7, 1e-3], T)
    off = np.array([0, T], dtype=np.int32)
    bg = np.ones(N)
    prob = X.Problem(context(), x, bg + 3.0, bg, off, pos, np.full(T, 0.5), c)
    phi = np.empty((S, 4, 1))
    phi[:, 0], phi[:, 3] = 1.0, 0.5
    phi[:, 1, 0] = [0.0, 0.0625, -0.03125, 0.01, 1e-9]
    phi[:, 2, 0] = [w, w, 2 * w, 0.0773, w]
    lo, hi = X.xrdvi_window_plan(context(), prob, dev(phi))
    rho = pos[None, :] + phi[:, 1]
    hw = c * phi[:, 2]
    want_lo = np.searchsorted(x, rho - hw, side="left")
    want_hi = np.maximum(np.searchsorted(x, rho + hw, side="right"), want_lo)
    assert np.array_equal(lo.cpu().numpy(), want_lo)
    assert np.array_equal(hi.cpu().numpy(), want_hi)
