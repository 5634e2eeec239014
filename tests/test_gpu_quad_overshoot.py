"""A first step that overshoots omega_f by many orders: the candidate state is
finite, its derivative is not.  The norm is then infinite and the step is
rejected, by four lanes on an inspiral as by one."""
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


def _spins(n, seed, top):
    """Masses 1 : 1 to 1 : 100, spins up to 10^top times the extreme one."""
    r = np.random.default_rng(seed)
    q = 10.0 ** r.uniform(0, 2, n)
    m = np.stack([q / (1 + q), 1 / (1 + q)])
    S = r.normal(size=(6, n))
    S[:3] *= m[0] ** 2 / np.linalg.norm(S[:3], axis=0)
    S[3:] *= m[1] ** 2 / np.linalg.norm(S[3:], axis=0)
    L = r.normal(size=(3, n))
    L /= np.linalg.norm(L, axis=0)
    w = 10.0 ** r.uniform(-2.2, -1.2, n)
    S *= 10.0 ** r.uniform(-3, top, n)
    return [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (m, S, L, w)]


@pytest.mark.parametrize("n,seed", [(1000, 6), (5200, 6), (16384, 3)])
def test_overshoot_equals_one_lane(n, seed):
    from paper_0908_3889_amd import api
    a = _spins(n, seed, 4)
    four = api.pn_integrate(*a, 0.05, 1e-7, api.make_opts(max_steps=900))
    one = api.pn_integrate(*a, 0.05, 1e-7, api.make_opts(max_steps=900, waves_per_simd=2))
    for k in ("status", "steps", "y", "t", "dots"):
        np.testing.assert_array_equal(four[k].cpu().numpy(), one[k].cpu().numpy(), err_msg=k)
    # the case is among them: inspirals whose first steps were rejected and
    # that then ran to omega_f
    st, steps = one["status"].cpu().numpy(), one["steps"].cpu().numpy()
    assert np.any((st == 0) & (steps[1] > 1))
