"""The density estimate where its products of exponentials end: bandwidths far
larger than the grid, infinite or negative, and points at the distance where
their last contribution to the grid vanishes, against the numpy definition of
oracle/stats.py."""
import numpy as np
import pytest

from oracle import stats as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# the bound of test_gpu_stats_paths.py, eps (3 u^2/2 + 16 |v d| + 40), with |u| <=
# 46 and |v d| <= 72: 4.9e-13, and the reference's own 3.5e-13; about twice both
RTOL = 2e-12


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import _lib
    _lib.load()
    yield


def _kde(x, sigma, ngrid, lo=-1.0, hi=1.0):
    from paper_0908_3889_amd import api
    return api.pn_kde(torch.from_numpy(np.stack([x])).cuda(), torch.tensor([sigma], dtype=torch.float64).cuda(), ngrid,
                      lo, hi).cpu().numpy()[0]


# n that is, and is not, a multiple of the points a wave takes at a time
@pytest.mark.parametrize("n", [1, 32, 33, 500])
@pytest.mark.parametrize("sigma", [1e3, 1e100, 1e280, 1e290, 1e300, 1e306, np.inf, -0.4, -3.0])
def test_kde_extreme_bandwidths(n, sigma):
    x = np.random.default_rng(n).uniform(-1.0, 1.0, n)
    for ngrid in (2, 201, 300):
        with np.errstate(over="ignore"):
            ref = S.kde(x, S.kde_grid(-1.0, 1.0, ngrid), 1.06 * sigma * n ** -0.2)
        got = _kde(x, sigma, ngrid)
        assert np.isfinite(ref).all()
        np.testing.assert_allclose(got, ref, rtol=RTOL, atol=0.0 if sigma < 1e306 else 1e-307)


# a grid step of d bandwidths, the points `away` bandwidths outside [lo, hi]
@pytest.mark.parametrize("d", [0.1, 0.3, 0.5, 0.58, 0.589999, 0.59, 0.590001, 0.6, 0.62, 0.7])
@pytest.mark.parametrize("away", [0.0, 20.0, 30.0, 34.0, 36.0, 37.0])
@pytest.mark.parametrize("ngrid", [9, 17, 25, 60, 95, 257, 300])
def test_kde_points_outside_the_grid(d, away, ngrid):
    sigma = (2.0 / (ngrid - 1)) / d / (1.06 * 3 ** -0.2)
    h = 1.06 * sigma * 3 ** -0.2
    for side in (-1.0, 1.0):
        x = side * (1.0 + h * (away + np.array([0.0, 0.21, 0.37])))
        ref = S.kde(x, S.kde_grid(-1.0, 1.0, ngrid), h)
        assert ref.max() > 1e-300
        np.testing.assert_allclose(_kde(x, sigma, ngrid), ref, rtol=RTOL, atol=1e-307)
