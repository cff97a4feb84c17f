"""Dense analyses of few peaks, every one taken at every point: both sides of the
rule (at most 48 phases; blocks of one sample T + K up to 128, of four 88,
asymmetric T + 2 K), in every kind of block, against the FP64 oracle: profile
1e-5, ELBO 1e-6, each phase's and latent's gradient 1e-4; served, the same bits
as alone."""
import pytest

from test_gpu_dense_few_phases import test_few_phases as check
from test_gpu_dense_few_phases import test_few_phases_served as check_served

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("asym,sec", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("N,S", [(1, 3), (64, 1), (900, 61), (700, 131), (1300, 202), (1409, 200)])
@pytest.mark.parametrize("M", [(87,), (88,), (127,), (128,), 48 * (1,), 49 * (1,), 44 * (1,),
                               45 * (1,), 29 * (1,), 30 * (1,), 47 * (0,) + (30,),
                               (30, 0, 50, 1), (3, 60, 22)],
                         ids=lambda m: f"{len(m)}x{m[0]}-{sum(m)}")
def test_few_peaks(M, N, S, asym, sec):
    check(M, N, S, asym, sec)


@pytest.mark.parametrize("M", [(60, 3, 20), 20 * (2,), (87, 1), (150, 3, 20)])
@pytest.mark.parametrize("N,S", [(700, 6), (900, 60), (700, 131), (1300, 200)])
def test_few_peaks_served(N, S, M):
    check_served(N, S, M)
