"""Call slots under load, on launches that take one: small FP64 batches at the
default options have a kernel that needs none, so these calls set waves_per_simd;
and the lists, which read their descriptor from the slot.  As test_gpu_slots.py:
more launches on two streams than the ring has slots (1024), graph replays beside
direct calls, each output equal bit for bit to an eager call's."""
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


def _same(out, ref, what):
    for k in ref:
        b = torch.int64 if ref[k].dtype == torch.float64 else torch.int32
        assert torch.equal(out[k].view(b), ref[k].view(b)), f"{what}: {k}"


def _fresh(api, n):
    out = api.alloc_outputs(n)
    for v in out.values():
        v.fill_(-77)
    return out


OPTS = [dict(waves_per_simd=2), dict(precision="fp32split"), dict(precision="fp32", block=64)]


def _small(n=192):
    from paper_0908_3889_amd import api
    pop = P.generate("adjoint_64k", n)          # three waves, short inspirals
    d = api.to_device(pop)
    return api, n, (d["m"], d["S"], d["L"], d["omega0"], pop["omega_f"], pop["tol"])


@pytest.mark.parametrize("kw", OPTS)
def test_launches_on_two_streams_beyond_the_ring(kw):
    api, n, a = _small()
    opts = api.make_opts(**kw)
    ref = api.pn_integrate(*a, opts, out=_fresh(api, n))
    outs = [[_fresh(api, n) for _ in range(600)] for _ in range(2)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for i in range(600):
        for s, pair in zip(streams, outs):
            api.pn_integrate(*a, opts, out=pair[i], stream=s)
    torch.cuda.synchronize()
    for j, pair in enumerate(outs):
        for i, o in enumerate(pair):
            _same(o, ref, f"stream {j} call {i}")


def _replays(api, a, n, opts, calls, every):
    """Replays of a captured call on one stream beside direct calls on another."""
    ref = api.pn_integrate(*a, opts, out=_fresh(api, n))
    gout, outs = _fresh(api, n), [_fresh(api, n) for _ in range(min(calls, 64))]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        api.pn_integrate(*a, opts, out=gout, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    main, rep = torch.cuda.Stream(), torch.cuda.Stream()
    for i in range(calls):
        api.pn_integrate(*a, opts, out=outs[i % len(outs)], stream=main)
        if i % every == every - 1:
            with torch.cuda.stream(rep):
                for v in gout.values():
                    v.fill_(-77)
                g.replay()
            rep.synchronize()
            _same(gout, ref, f"replay after direct call {i}")
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        _same(o, ref, f"direct call {i}")


@pytest.mark.parametrize("kw", OPTS)
def test_replays_beside_more_direct_calls_than_the_ring_holds(kw):
    api, n, a = _small()
    _replays(api, a, n, api.make_opts(**kw), 1100, 100)


# one more inspiral than a wave on each SIMD holds: the lists; without an order,
# with pn_cost_order's and records, with another order and records
@pytest.mark.parametrize("order", [None, "cost", "other"])
@pytest.mark.parametrize("precision", ["fp64", "fp32split"])
def test_lists_replayed_beside_direct_lists(precision, order):
    from paper_0908_3889_amd import api
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 256 * cus + 1
    pop = P.generate("adjoint_64k", 4096)
    d = api.to_device(pop)
    m, S, L, w = (d[k].repeat(*([1] * (d[k].dim() - 1)), n // 4096 + 1)[..., :n].contiguous()
                  for k in ("m", "S", "L", "omega0"))
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    w.copy_(0.03 + 0.018 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64))
    a = (m, S, L, w, 0.05, 1e-6)
    kw = {}
    if order:
        kw["packed"] = api.packed_inputs(n)
        kw["order"] = api.pn_cost_order(*a[:5], packed=kw["packed"])
        if order == "other":
            kw["order"] = torch.randperm(n, generator=g, device="cuda").to(torch.int32)
    _replays(api, a, n, api.make_opts(precision=precision, **kw), 24, 6)
