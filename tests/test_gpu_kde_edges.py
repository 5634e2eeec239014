"""The density estimate where its products of exponentials end: bandwidths far
larger than the grid, infinite or negative, against the numpy definition of
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
