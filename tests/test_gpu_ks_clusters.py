"""The K-S statistic of samples whose values cluster in a few of the buckets it
counts in: ties, narrow clusters, values outside the interval.  D is the sorted
sample's bit for bit, and takes a few times a spread sample's time, not that of
one block reading the sample over and over."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import _lib
    _lib.load()
    yield


def _sample(kind, n, seed):
    rng = np.random.default_rng(seed)
    u = rng.uniform(-1.0, 1.0, n)
    if kind == "uniform":
        return u
    if kind == "one value":
        return np.full(n, 0.25)
    if kind == "two values":
        return np.where(u < 0.1, -0.3, 0.4)
    if kind == "a third at zero":                     # a spin of zero, and signed zeros
        return np.where(u < -0.33, np.where(rng.random(n) < 0.5, 0.0, -0.0), rng.uniform(-1.0, 1.0, n))
    if kind == "half at the end":                     # aligned spins: 1, or 1 less a few ulp
        return np.where(u < 0.0, 1.0 - 1.1102230246251565e-16 * rng.integers(0, 3, n), rng.uniform(-1.0, 1.0, n))
    if kind == "nearly aligned":                      # all within 1e-8 of 1
        return 1.0 - 1e-8 * u * u
    if kind == "fourteen clusters":
        return (rng.integers(0, 14, n) - 7) / 7.5 + 1e-9 * u
    if kind == "clusters in clusters":                # at three scales about one value
        return 0.2 + u * np.array([1e-4, 1e-9, 1e-14, 0.0])[rng.integers(0, 4, n)]
    if kind == "outside":
        return np.where(rng.random(n) < 0.6, 3.0 * u, 1e5 * u)
    if kind == "infinite":
        return np.where(rng.random(n) < 0.5, np.where(u < 0.2, -np.inf, np.inf), u)
    if kind == "periodic":                            # a cluster, and one place in 256 (or n / 16384) elsewhere
        x = 0.6 + 1e-10 * u
        x[::max(2, n // 16384)] = rng.uniform(-1.0, 0.0, x[::max(2, n // 16384)].size)
        return x
    raise ValueError(kind)


KINDS = ["one value", "two values", "a third at zero", "half at the end", "nearly aligned", "fourteen clusters",
         "clusters in clusters", "outside", "infinite", "periodic"]


def _ks_D(x, lo=-1.0, hi=1.0):
    """The definition on the sorted values, every operation rounded as written."""
    xs = np.sort(x)
    n = float(xs.size)
    i = np.arange(xs.size, dtype=np.float64)
    F = (xs - lo) / (hi - lo)
    return max(0.0, np.max((i + 1.0) / n - F), np.max(F - i / n))


# one block; a bucket of 4096 values and one more; two blocks and a ragged one;
# sizes at which all splitters are used
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [16384, 16385, 40000, 65537, 300001, 1 << 20])
def test_ks_of_clusters_is_the_sorted_samples(kind, n):
    from paper_0908_3889_amd import api
    x = np.stack([_sample(kind, n, n + c) for c in range(3)])
    x[1] = np.sort(x[1])
    got = api.pn_ks_uniform(torch.from_numpy(x).cuda()).cpu().numpy()
    assert list(got[:, 0]) == [_ks_D(c) for c in x]


@pytest.mark.parametrize("m", [4095, 4096, 4097, 4128])
def test_ks_at_the_smallest_split_bucket(m):
    from paper_0908_3889_amd import api
    n = 50000
    x = np.random.default_rng(m).uniform(-1.0, 1.0, n)
    x[np.abs(x - 0.3) < 1e-3] = 0.9
    x[:m] = 0.3 + 1e-12 * np.arange(m)
    x = np.random.default_rng(m + 1).permutation(x)
    assert float(api.pn_ks_uniform(torch.from_numpy(x).cuda())[0, 0]) == _ks_D(x)


# 3 to 41 times a spread sample's time when one block refined a bucket alone
# (2^16 .. 2^22 values); a sort of all values takes 2 to 4 times
@pytest.mark.parametrize("kind", KINDS)
def test_time_of_clusters(kind):
    from paper_0908_3889_amd import api
    n = 1 << 22

    def ms(x):
        t = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            api.pn_ks_uniform(x)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    spread = ms(torch.from_numpy(_sample("uniform", n, 1)).cuda())
    clusters = ms(torch.from_numpy(_sample(kind, n, 2)).cuda())
    print(f"\n{kind}: {clusters:.3f} ms, uniform {spread:.3f} ms", flush=True)
    assert clusters < 5.0 * spread
