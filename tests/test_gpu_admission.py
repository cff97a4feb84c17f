"""Admission of analyses to a running server: one copy from staging memory.

The staging buffers alternate and grow, so analyses of growing and shrinking
sizes enter back to back; a phase without peaks, unsorted peak positions and a
single step are the sizes at which the staged image can go wrong.  The served
result is the one-at-a-time runner's (the bar of the other serving tests).
"""
import numpy as np
import pytest

from paper_2501_09308_amd import xrdvi as X
from gpu_common import context
from test_gpu_serving import wait_all

pytestmark = pytest.mark.gpu


class _Req:
    def __init__(self, rng, N, K, m, cutoff, order):
        self.x = 10.0 + 0.02 * np.arange(N)
        self.bg = 5.0 + rng.random(N)
        self.cutoff = cutoff
        self.y = np.floor(self.bg + 10.0 + 50.0 * rng.random(N))
        counts = np.full(K, m)
        counts[K // 2] = 0 if K > 1 else m
        self.peak_off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
        parts = []
        for c in counts:
            p = rng.uniform(self.x[0], self.x[-1] + 1e-9, c)
            parts.append(np.sort(p) if order == "sorted" else np.sort(p)[::-1] if order == "reversed" else p)
        self.peak_pos = np.concatenate(parts)
        self.peak_int = rng.random(self.peak_pos.size)


@pytest.mark.parametrize("order", ["sorted", "reversed", "shuffled"])
def test_sizes_that_grow_and_shrink_back_to_back(order):
    rng = np.random.default_rng(5)
    sizes = [(1, 1, 1, 8.0, 1), (700, 3, 5, 0.0, 6), (3001, 40, 30, 8.0, 11), (2, 2, 1, 0.0, 1),
             (5000, 90, 25, 6.0, 7), (130, 1, 2, 8.0, 12), (1025, 17, 9, 0.0, 3)]
    reqs = [(_Req(rng, N, K, m, c, order), steps) for N, K, m, c, steps in sizes]
    srv = X.Server(arena_bytes=256 << 20, max_slots=4, steps_per_launch=5)
    tickets = [srv.submit(r, r.y, 3, steps, 40 + i) for i, (r, steps) in enumerate(reqs)]
    res = wait_all(srv, tickets)
    srv.close()
    ctx = context()
    for i, (r, steps) in enumerate(reqs):
        rc, info, out = res[tickets[i]]
        assert rc == X.XRDVI_OK
        ref = X.xrdvi_plain_run(ctx, r, r.y, 3, steps, 40 + i)
        for k in ("loc", "logscale", "trace"):
            np.testing.assert_allclose(out[k], ref[k], rtol=1e-12, atol=1e-12)
