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


def _ks_sample(kind, n, seed):
    rng = np.random.default_rng(seed)
    u = rng.uniform(-1.0, 1.0, n)
    if kind == "uniform":
        return u
    if kind == "normal":
        return np.clip(rng.normal(0.1, 0.4, n), -1.0, 1.0)
    if kind == "constant":
        return np.full(n, 0.25)
    if kind == "half at the end":                    # aligned spins: 1, or 1 less a few ulp
        return np.where(rng.random(n) < 0.5, 1.0 - 1.1102230246251565e-16 * rng.integers(0, 3, n), u)
    if kind == "cluster":                            # far narrower than a bucket
        return np.where(rng.random(n) < 0.7, 0.3 + 1e-9 * u, u)
    if kind == "cluster at zero":                    # keys over the whole exponent range
        return np.where(rng.random(n) < 0.7, u * 10.0 ** rng.uniform(-300, -5, n), u)
    if kind == "ties":
        return np.round(u * 50.0) / 50.0
    if kind == "outside":                            # the first and last bucket hold far values
        return np.where(rng.random(n) < 0.6, 3.0 * u, 1e5 * u)
    raise ValueError(kind)


def _ks_D(x, lo=-1.0, hi=1.0):
    """The definition on the sorted values, every operation rounded as written."""
    xs = np.sort(x)
    n = float(xs.size)
    i = np.arange(xs.size, dtype=np.float64)
    F = (xs - lo) / (hi - lo)
    return max(0.0, np.max((i + 1.0) / n - F), np.max(F - i / n))


KS_KINDS = ["uniform", "normal", "constant", "half at the end", "cluster", "cluster at zero", "ties", "outside"]


# D is a maximum of rounded values, taken over the same values: equal bit for bit
@pytest.mark.parametrize("kind", KS_KINDS)
@pytest.mark.parametrize("n", [1, 2, 65, 1024, 4099, 16384, 16385, 70001])
def test_ks_is_the_sorted_samples(kind, n):
    x = np.stack([_ks_sample(kind, n, 7 * n + c) for c in range(3)])
    got = _api().pn_ks_uniform(_cuda(x)).cpu().numpy()
    for c in range(3):
        assert got[c, 0] == _ks_D(x[c])
        np.testing.assert_allclose(got[c, 1], S.ks_uniform(x[c], -1.0, 1.0)["p"], rtol=1e-12, atol=1e-300)


@pytest.mark.parametrize("n", [1 << 20, (1 << 22) - 3, 1 << 22, (1 << 22) + 1])
def test_ks_at_the_largest_bucketed_size(n):
    for kind in ("uniform", "normal"):
        x = _ks_sample(kind, n, n + 1)
        assert _api().pn_ks_uniform(_cuda(x)).cpu().numpy()[0, 0] == _ks_D(x)


def test_ks_other_interval_and_workspaces():
    import ctypes as C

    from paper_0908_3889_amd import _lib
    L = _lib.load()
    n, nc, lo, hi = 40000, 5, -0.7, 1.9
    x = np.stack([_ks_sample(k, n, 3) for k in KS_KINDS[:nc]])
    xt = _cuda(x)
    full = int(L.pn_ks_workspace_bytes(n))
    p = lambda t: C.c_void_p(t.data_ptr())
    # three, two and one components side by side
    for ws_bytes in (full, full * 2 // 3, full * 5 // 9):
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
        out = torch.empty((nc, 2), dtype=torch.float64, device="cuda")
        _lib.check(L.pn_ks_uniform(n, n, p(xt), nc, lo, hi, p(out), p(ws), ws_bytes, None), "pn_ks_uniform")
        torch.cuda.synchronize()
        assert [float(v) for v in out[:, 0].cpu()] == [_ks_D(x[c], lo, hi) for c in range(nc)]
    out = torch.empty((nc, 2), dtype=torch.float64, device="cuda")
    assert L.pn_ks_uniform(n, n, p(xt), nc, lo, hi, p(out), p(ws), 1024, None) == _lib.PN_EINVAL


# one block, the first size of two, a ragged last one; bins from one copy of the
# counters to 32; values on the edges, outside and not a number; a leading
# dimension above n
@pytest.mark.parametrize("n", [1, 1000, 16384, 16385, 50001])
@pytest.mark.parametrize("nbins", [1, 20, 79, 128])
def test_histogram_blocks(n, nbins):
    api = _api()
    rng = np.random.default_rng(n + nbins)
    lo, hi = -1.0, 0.9
    x = rng.uniform(-1.1, 1.1, (2, n))
    edges = S.bin_edges(lo, hi, nbins)
    k = min(n, edges.size)
    x[0, :k] = edges[:k]
    if n > 1:
        x[1, -1] = np.nan
    y = np.roll(x, 1, axis=1) * 0.9
    wide = torch.zeros((4, n + 13), dtype=torch.float64, device="cuda")
    wide[:2, :n], wide[2:, :n] = _cuda(x), _cuda(y)
    one = api.pn_histogram(wide[:2, :n], nbins, lo, hi).cpu().numpy()
    two = api.pn_histogram2d(wide[:2, :n], wide[2:, :n], nbins, lo, hi).cpu().numpy()
    for c in range(2):
        assert (one[c] == S.histogram(x[c], lo, hi, nbins)).all()
        assert (two[c] == S.histogram2d(x[c], y[c], lo, hi, nbins)).all()


def test_histogram_largest_number_of_bins():
    x = np.random.default_rng(9).uniform(-1.0, 1.0, (1, 30000))
    for nbins in (129, 256, 2048, 4096):
        assert (_api().pn_histogram(_cuda(x), nbins).cpu().numpy()[0] == S.histogram(x[0], -1.0, 1.0, nbins)).all()


# bins so narrow against the interval's ends that the rounding of an edge is a
# good part of a bin: every value is placed by the edges
def test_histogram_bins_near_the_rounding_of_the_edges():
    lo, hi, nbins = 1e10, 1e10 + 1e-4, 20
    x = np.random.default_rng(4).uniform(lo, hi, (1, 20000))
    assert (_api().pn_histogram(_cuda(x), nbins, lo, hi).cpu().numpy()[0] == S.histogram(x[0], lo, hi, nbins)).all()


# one block, the first size of two passes, and sizes around the blocks of a pass;
# a large common offset, which one pass of raw moments would lose.  Bounds: the
# sums of n terms in trees of depth about log2 n + 16, so 64 eps of the sum of
# magnitudes, which for the centred sums is the sum itself; the mean's error
# enters the centred sums squared.
@pytest.mark.parametrize("n", [2, 63, 1024, 16383, 16384, 16385, 131072, 131073, 300001])
def test_pearson_blocks(n):
    rng = np.random.default_rng(n)
    x = rng.normal(0.0, 1.0, (3, n)) + np.array([[0.0], [1e3], [-7.0]])
    y = 0.6 * x + rng.normal(0.0, 0.8, (3, n))
    wide = torch.zeros((6, n + 5), dtype=torch.float64, device="cuda")
    wide[:3, :n], wide[3:, :n] = _cuda(x), _cuda(y)
    got = _api().pn_pearson(wide[:3, :n], wide[3:, :n]).cpu().numpy()
    eps = 2.0 ** -52
    for c in range(3):
        xl, yl = x[c].astype(np.longdouble), y[c].astype(np.longdouble)
        mx, my = xl.mean(), yl.mean()
        sx, sy = ((xl - mx) ** 2).sum(), ((yl - my) ** 2).sum()
        r = ((xl - mx) * (yl - my)).sum() / np.sqrt(sx * sy)
        scale = np.abs(x[c]).max() + np.abs(y[c]).max()      # a centred value's rounding: eps of this
        slack = 64 * eps + 4 * eps * scale / min(np.sqrt(sx / n), np.sqrt(sy / n))
        assert abs(got[c, 0] - mx) <= 64 * eps * np.abs(x[c]).mean()
        assert abs(got[c, 1] - my) <= 64 * eps * np.abs(y[c]).mean()
        assert abs(got[c, 2] / np.sqrt(sx / (n - 1)) - 1) <= slack
        assert abs(got[c, 3] / np.sqrt(sy / (n - 1)) - 1) <= slack
        assert abs(got[c, 4] - r) <= slack


# more chunks of 4,096 values than blocks: the same bounds (the combined sums
# add one more level)
@pytest.mark.parametrize("n", [1048576, 1048577, 1052673, 2100003])
def test_pearson_chunks(n):
    test_pearson_blocks(n)
