"""pn_generate at the edges of its 256-inspiral blocks, whose spheres without
an accepted first attempt are drawn on by other lanes: bit for bit the
oracle's draws."""
import numpy as np
import pytest

from oracle import generate as G

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import _lib
    _lib.load()
    yield


@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 1000, 100003])
@pytest.mark.parametrize("seed,first", [(1, 0), (2 ** 63 + 12345, 2 ** 41 + 7)])
def test_blocks_bit_exact(n, seed, first):
    from paper_0908_3889_amd import api
    spec = api.gen_spec((1.0, 4.0), (0.1, 0.9), (0.0, 1.0), (0.004, 0.01), seed=seed)
    got = api.pn_generate(n, spec, first)
    ref = G.population(n, seed, ("uniform", 1.0, 4.0), ("uniform", 0.0, 1.0), ("uniform", 0.004, 0.01), first=first)
    for k in ("m", "L", "omega0"):
        np.testing.assert_array_equal(got[k].cpu().numpy(), ref[k], err_msg=k)
    # the oracle draws both Kerr parameters from one range; take the second spin, and the directions of both
    S, R = got["S"].cpu().numpy(), ref["S"]
    np.testing.assert_array_equal(S[3:], R[3:])
    np.testing.assert_allclose(S[:3] / np.linalg.norm(S[:3], axis=0), R[:3] / np.linalg.norm(R[:3], axis=0), rtol=0,
                               atol=1e-15)
