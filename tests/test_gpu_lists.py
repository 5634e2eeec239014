"""Calls without an order that put more than one wave on a SIMD share the
inspirals out to the CUs, longest first in each.  A call that sets
waves_per_simd takes them as they come; each inspiral's results are equal bit
for bit."""
import numpy as np
import pytest

from paper_0908_3889_amd import population as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import _lib
    _lib.load()
    yield


WAVES = {"fp64": 2, "fp32split": 3, "fp32": 3}


# the edges of the range on 256 CUs (65,536 < n <= 2,097,152), of a list's full
# waves (131,072 and 196,608), odd sizes, and rows of more columns than n
SIZES = (65536, 65537, 67583, 100003, 131072, 131073, 196609, 500009, 1048577, 2097152, 2097153)


@pytest.mark.parametrize("n,phase", [(n, False) for n in SIZES] + [(67583, True), (131073, True)])
@pytest.mark.parametrize("precision", ["fp64", "fp32split", "fp32"])
def test_lists_equal_as_they_come(n, precision, phase):
    from paper_0908_3889_amd import api
    ld = n + 5
    pop = P.generate("q1to4_1M", 4096)
    d = {}
    for k in ("m", "S", "L", "omega0"):
        full = torch.from_numpy(pop[k]).to("cuda").repeat(*([1] * (pop[k].ndim - 1)), ld // 4096 + 1)
        d[k] = full[..., :ld].contiguous()[..., :n]
    # short inspirals of different lengths, and every outcome at odd places
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    d["omega0"].copy_(0.03 + 0.015 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64))
    d["m"][0, 3::1999] = -1.0
    d["S"][2, 5::2001] = float("nan")
    d["omega0"][7::777] = 0.05
    d["S"][:, 11::1501] = 0.0
    d["omega0"][n - 1] = 0.025
    a = (d["m"], d["S"], d["L"], d["omega0"], 0.05, 1e-6)
    call = api.pn_integrate_phase if phase else api.pn_integrate

    def result(**kw):
        out = {k: torch.full_like(v, -5)[..., :n] for k, v in api.alloc_outputs(ld).items()}
        return call(*a, api.make_opts(precision=precision, **kw), out=out)

    def same(x, y):
        assert x.keys() == y.keys()
        for k in x:
            b = torch.int64 if x[k].dtype == torch.float64 else torch.int32
            assert torch.equal(x[k].view(b), y[k].view(b)), k

    x, y = result(), result(waves_per_simd=WAVES[precision])
    same(x, y)
    if n == 100003:      # a hand-out order with packed records, entries of it that are no index or there twice
        packed = api.packed_inputs(n)
        order = api.pn_cost_order(*a[:5], packed=packed)
        same(result(order=order, packed=packed), y)
        same(result(packed=packed), y)
        order[4], order[50], order[n - 1] = -1, n, order[60]
        same(*(result(order=order, packed=packed, **kw) for kw in ({}, {"waves_per_simd": WAVES[precision]})))
    st = np.unique(x["status"].cpu().numpy())
    assert len(st) >= 3
