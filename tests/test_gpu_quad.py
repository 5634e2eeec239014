"""Small FP64 batches run four lanes on one inspiral; larger ones, and any
call that sets waves_per_simd, one.  Both form every number by the same
operations, so their results are equal bit for bit."""
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


def _api():
    from paper_0908_3889_amd import api
    return api


def _args(pop):
    d = _api().to_device(pop)
    return (d["m"], d["S"], d["L"], d["omega0"], pop["omega_f"], pop["tol"])


def _equal(a, b, keys):
    for k in keys:
        x, y = a[k].cpu().numpy(), b[k].cpu().numpy()
        np.testing.assert_array_equal(x, y, err_msg=k)


KEYS = ("y", "t", "steps", "status", "dots")


@pytest.mark.parametrize("workload", ["q1to4_1M", "batching_4M", "equal_mass_maxspin_1k", "paper_equal_mass"])
@pytest.mark.parametrize("n", [1, 3, 15, 16, 17, 1000, 16384, 16385])
def test_four_lanes_equal_one(workload, n):
    api = _api()
    a = _args(P.generate(workload, n))
    _equal(api.pn_integrate(*a), api.pn_integrate(*a, api.make_opts(waves_per_simd=2)), KEYS)


@pytest.mark.parametrize("n", [1, 17, 500])
def test_phase_and_tape_equal(n):
    api = _api()
    a = _args(P.generate("q1to4_1M", n))
    one = api.make_opts(waves_per_simd=2)
    _equal(api.pn_integrate_phase(*a), api.pn_integrate_phase(*a, one), KEYS + ("phase",))
    for every in (1, 16, 64):
        r, s = (api.pn_integrate_record(*a, o, cap_steps=1024, ckpt_every=every) for o in (None, one))
        _equal(r, s, KEYS)
        acc = r["steps"][0].cpu().numpy()
        tr, ts = r["tape"].cpu().numpy(), s["tape"].cpu().numpy()
        np.testing.assert_array_equal(tr[:, :2], ts[:, :2])
        for i in range(n):
            np.testing.assert_array_equal(tr[i, 2:2 + acc[i]], ts[i, 2:2 + acc[i]])
            c = slice(2 + 1024, 2 + 1024 + 10 * (acc[i] // every + 1))
            np.testing.assert_array_equal(tr[i, c], ts[i, c])


# every outcome of an inspiral, options that change the equations, a hand-out
# order with entries that are no index, packed records
def test_outcomes_and_options():
    api = _api()
    n = 100
    pop = P.generate("q1to4_1M", n)
    pop["m"][0, 3] = -1.0
    pop["S"][2, 5] = np.nan
    pop["omega0"][7] = pop["omega_f"]
    pop["omega0"][9] = pop["omega_f"] * (1 - 1e-9)
    pop["S"][:, 11] = 0.0
    pop["S"][3:, 13] = 0.0
    pop["omega0"][15] = 3.0e3                 # above omega_f
    pop["S"][:, 17] *= 1e3                    # d omega/dt <= 0 on the way
    a = _args(pop)
    for kw in ({}, {"max_steps": 40}, {"terms": 8}, {"terms": 63 & ~8, "max_steps": 50}, {"theta_literal": 1}, {"h0": 1e4},
               {"h0": 1e-9}, {"max_steps": 1}):
        x = api.pn_integrate(*a, api.make_opts(**kw))
        y = api.pn_integrate(*a, api.make_opts(waves_per_simd=2, **kw))
        _equal(x, y, KEYS)
    r, s = (api.pn_integrate_record(*a, o, cap_steps=60, ckpt_every=16) for o in
            (None, api.make_opts(waves_per_simd=2)))
    _equal(r, s, KEYS)
    packed = api.packed_inputs(n)
    order = api.pn_cost_order(*a[:5], packed=packed)
    _equal(api.pn_integrate(*a), api.pn_integrate(*a, api.make_opts(order=order, packed=packed)), KEYS)
    order[4] = -1
    order[50] = n
    out, ref = ({k: torch.full_like(v, -5) for k, v in api.alloc_outputs(n).items()} for _ in range(2))
    api.pn_integrate(*a, api.make_opts(order=order), out=out)
    api.pn_integrate(*a, api.make_opts(order=order, waves_per_simd=2), out=ref)
    _equal(out, ref, KEYS)


# tolerances at which a product of error scales leaves the normal range
@pytest.mark.parametrize("tol", [1e-3, 1e-13, 1e-80, 1e-110, 1e200])
def test_extreme_tolerances(tol):
    api = _api()
    a = _args(P.generate("adjoint_64k", 64))[:5] + (tol,)
    kw = {"max_steps": 200}
    _equal(api.pn_integrate(*a, api.make_opts(**kw)), api.pn_integrate(*a, api.make_opts(waves_per_simd=2, **kw)), KEYS)
