"""A hand-out order that comes with packed records: pn_cost_order's is refined by
the lists, any other is kept, as it is without the records.  Results do not depend
on it; the speed of an order by the true numbers of steps does."""
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


def _equal_masses(n, omega0, seed):
    """m1 = m2, maximal isotropic spins, L_hat = z: (m, S, L, omega0) on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    S = torch.randn(2, 3, n, generator=g, device="cuda", dtype=torch.float64)
    S = (0.25 * S / S.norm(dim=1, keepdim=True)).reshape(6, n)
    L = torch.zeros(3, n, device="cuda", dtype=torch.float64)
    L[2] = 1.0
    return (torch.full((2, n), 0.5, device="cuda", dtype=torch.float64), S, L,
            torch.full((n,), omega0, device="cuda", dtype=torch.float64))


@pytest.mark.parametrize("precision", ["fp64", "fp32split", "fp32"])
@pytest.mark.parametrize("entry", ["plain", "phase", "noalloc"])
def test_results_do_not_depend_on_the_order(precision, entry):
    from paper_0908_3889_amd import api
    n = 70001
    a = _equal_masses(n, 0.03, 1) + (0.05,)
    packed = api.packed_inputs(n)
    cost = api.pn_cost_order(*a, packed=packed)
    call = {"plain": api.pn_integrate, "phase": api.pn_integrate_phase, "noalloc": api.pn_integrate_noalloc}[entry]

    def run(**kw):
        out = api.alloc_outputs(n)
        if entry == "phase":
            out["phase"] = torch.empty(n, device="cuda", dtype=torch.float64)
        for v in out.values():
            v.fill_(-77)
        return call(*a, 1e-6, opts=api.make_opts(precision=precision, **kw), out=out)

    ref = run()
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    for order in (cost, torch.argsort(ref["steps"][0], descending=True).to(torch.int32), cost.flip(0).contiguous(),
                  torch.randperm(n, generator=g, device="cuda").to(torch.int32)):
        for records in (packed, None):
            out = run(order=order, packed=records)
            for k in ref:
                b = torch.int64 if ref[k].dtype == torch.float64 else torch.int32
                assert torch.equal(out[k].view(b), ref[k].view(b)), k
    # entries that are no index at the places looked at, and everywhere
    bad = cost.clone()
    bad[0], bad[(n - 1) * 20 // 63], bad[n - 1] = -1, n, -5
    for order in (bad, torch.full_like(cost, -1)):
        out = run(order=order, packed=packed)
        keep = order[(order >= 0) & (order < n)].long()
        gone = torch.ones(n, dtype=torch.bool, device="cuda")
        gone[keep] = False
        assert torch.equal(out["y"][:, keep], ref["y"][:, keep])
        assert (out["status"][gone] == -77).all()


# by the true numbers of steps the records' order took 1.21 times the order's time
# while the lists ranked it anew
@pytest.mark.parametrize("precision", ["fp64", "fp32split"])
def test_time_of_an_order_by_the_true_steps(precision):
    from paper_0908_3889_amd import api
    n = 1 << 20
    a = _equal_masses(n, 0.00395, 3) + (0.05,)
    packed, out = api.packed_inputs(n), api.alloc_outputs(n)
    api.pn_cost_order(*a, packed=packed)
    api.pn_integrate(*a, 5e-7, api.make_opts(precision=precision), out=out)
    order = torch.argsort(out["steps"][0] + out["steps"][1], descending=True).to(torch.int32)

    opts = [api.make_opts(precision=precision, order=order, **kw) for kw in ({}, dict(packed=packed))]
    best = [1e9, 1e9]
    for _ in range(8):                                # in turn
        for i, o in enumerate(opts):
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s.record()
            api.pn_integrate(*a, 5e-7, o, out=out)
            e.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], s.elapsed_time(e))
    alone, records = best
    print(f"\n{precision}: {alone:.3f} ms, with records {records:.3f} ms", flush=True)
    assert records < 1.08 * alone
