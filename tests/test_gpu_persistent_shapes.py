"""The persistent kernels in each launch shape on small batches, which take a kernel
of their own unless waves_per_simd is set: the shapes against the static schedule,
equal bit for bit."""
import numpy as np
import pytest

from paper_0908_3889_amd import population as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("y", "t", "steps", "status", "dots")
SHAPES = [dict(block=b, waves_per_simd=w, refill_min=r) for b, w, r in
          ((64, 2, 0), (128, 1, 1), (256, 2, 8), (512, 2, 64), (64, 4, 3), (128, 2, 0), (512, 1, 1))]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import _lib
    _lib.load()
    yield


def _args(workload, n):
    from paper_0908_3889_amd import api
    pop = P.generate(workload, n)
    d = api.to_device(pop)
    return api, (d["m"], d["S"], d["L"], d["omega0"], pop["omega_f"], pop["tol"])


def _same(a, b, keys, what):
    for k in keys:
        np.testing.assert_array_equal(a[k].cpu().numpy(), b[k].cpu().numpy(), err_msg=f"{what} {k}")


@pytest.mark.parametrize("precision", ["fp64", "fp32split", "fp32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_shapes_equal_the_static_schedule(precision, shape):
    api, a = _args("batching_4M", 3001)
    base = api.pn_integrate_phase(*a, api.make_opts(precision=precision, schedule="static"))
    opts = api.make_opts(precision=precision, **shape)
    _same(api.pn_integrate(*a, opts), base, KEYS, shape)
    _same(api.pn_integrate_phase(*a, opts), base, KEYS + ("phase",), shape)


@pytest.mark.parametrize("shape", SHAPES)
def test_recorded_tapes_equal_the_static_schedules(shape):
    api, a = _args("batching_4M", 333)
    K, cap = 16, 4096
    base, rec = (api.pn_integrate_record(*a, api.make_opts(**kw), cap_steps=cap, ckpt_every=K)
                 for kw in (dict(schedule="static"), shape))
    _same(rec, base, KEYS, shape)
    for x, y, N in zip(rec["tape"].cpu().numpy(), base["tape"].cpu().numpy(), base["steps"][0].cpu().numpy()):
        np.testing.assert_array_equal(x[:2 + N], y[:2 + N])
        c = slice(2 + cap, 2 + cap + 10 * (N // K + 1))
        np.testing.assert_array_equal(x[c], y[c])


# the no-allocation entry point on its scratch: the second call smaller, queued
# behind the first
@pytest.mark.parametrize("kw", [dict(waves_per_simd=2), dict(waves_per_simd=2, block=64), dict(precision="fp32")])
def test_noalloc_on_the_persistent_grid(kw):
    api, a = _args("q1to4_1M", 3001)
    opts = api.make_opts(**kw)
    outs, refs = [], []
    for n in (3001, 1000):
        sub = tuple(t[..., :n].contiguous() for t in a[:4]) + a[4:]
        refs.append(api.pn_integrate(*sub, api.make_opts(schedule="static", precision=kw.get("precision", "fp64"))))
        outs.append({k: v.fill_(-77) for k, v in api.alloc_outputs(n).items()})
        api.pn_integrate_noalloc(*sub, outs[-1], opts)
    torch.cuda.synchronize()
    for out, ref in zip(outs, refs):
        _same(out, ref, KEYS, kw)


# hand-out orders, and the sizes on both sides of the four-lane kernel's range
@pytest.mark.parametrize("n", [3001, 16384, 16385])
def test_orders_and_sizes_equal_the_static_schedule(n):
    api, a = _args("q1to4_1M", n)
    base = api.pn_integrate(*a, api.make_opts(schedule="static"))
    order = torch.from_numpy(np.random.default_rng(n).permutation(n).astype(np.int32)).cuda()
    for kw in ({}, dict(waves_per_simd=2), dict(order=order), dict(order=order, waves_per_simd=2)):
        _same(api.pn_integrate(*a, api.make_opts(**kw)), base, KEYS, kw.keys())
