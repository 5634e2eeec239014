"""The statistics kernels at the edges of their tiles and dispatch rules,
against the numpy definitions of oracle/stats.py."""
import numpy as np
import pytest

from oracle import stats as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import _lib
    _lib.load()
    yield


def _api():
    from paper_0908_3889_amd import api
    return api


def _values(n, seed, ncomp=1):
    rng = np.random.default_rng(seed)
    return np.clip(np.stack([rng.normal(0.1 * c, 0.4, n) for c in range(ncomp)]), -1.0, 1.0)


def _cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# A density value is a sum of positive terms exp(-u^2/2).  A term's relative
# error is at most eps (3 u^2/2 + 16 |v d| + 40) with |u| <= 45, |v d| <= 37
# (the argument's rounding, its products, the polynomial): 4e-13, and the
# reference's own is 3 u^2/2 eps; the bound below is about four times both.
KDE_RTOL = 2e-12


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 4099])
@pytest.mark.parametrize("ngrid", [2, 15, 16, 17, 201, 255, 256, 257, 513])
def test_kde_tiles(n, ngrid):
    x = _values(n, n * 1000 + ngrid, 2)
    sigma = np.array([0.45, 0.3])
    got = _api().pn_kde(_cuda(x), _cuda(sigma), ngrid).cpu().numpy()
    grid = S.kde_grid(-1.0, 1.0, ngrid)
    for c in range(2):
        ref = S.kde(x[c], grid, 1.06 * sigma[c] * n ** -0.2)
        np.testing.assert_allclose(got[c], ref, rtol=KDE_RTOL, atol=1e-307)


# bandwidths on both sides of the rule (step against bandwidth, range against
# bandwidth), and densities down to the smallest a double holds
@pytest.mark.parametrize("sigma", [3.0, 0.3, 0.05, 0.02, 0.011, 0.0109, 0.01, 1e-3, 1e-6])
def test_kde_bandwidths(sigma):
    n, ngrid = 1000, 401
    x = 0.2 + 0.02 * _values(n, 5)
    got = _api().pn_kde(_cuda(x), _cuda(np.array([sigma])), ngrid).cpu().numpy()
    ref = S.kde(x[0], S.kde_grid(-1.0, 1.0, ngrid), 1.06 * sigma * n ** -0.2)
    np.testing.assert_allclose(got[0], ref, rtol=KDE_RTOL, atol=1e-307)


def test_kde_outliers_and_nonfinite_values():
    api = _api()
    n, ngrid = 500, 201
    x = _values(n, 6)
    x[0, [3, 70, 499]] = [1e6, -1e300, 40.0]          # far outside the grid: no contribution
    grid = S.kde_grid(-1.0, 1.0, ngrid)
    sig = _cuda(np.array([0.4]))
    ref = S.kde(x[0], grid, 1.06 * 0.4 * n ** -0.2)
    np.testing.assert_allclose(api.pn_kde(_cuda(x), sig, ngrid).cpu().numpy()[0], ref, rtol=KDE_RTOL, atol=1e-307)
    x[0, [3, 70, 499]] = [np.inf, -np.inf, np.inf]
    np.testing.assert_allclose(api.pn_kde(_cuda(x), sig, ngrid).cpu().numpy()[0], ref, rtol=KDE_RTOL, atol=1e-307)
    x[0, 130] = np.nan                                # a value that is not a number: no density
    assert np.isnan(api.pn_kde(_cuda(x), sig, ngrid).cpu().numpy()).all()
    for s in (0.0, np.nan):                           # nor with such a bandwidth
        assert np.isnan(api.pn_kde(_cuda(_values(n, 6)), _cuda(np.array([s])), ngrid).cpu().numpy()).all()
