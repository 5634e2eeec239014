"""Small batches reverse the steps of an inspiral in parts side by side; with
the workspace of one segment per inspiral alone, and in larger batches, one
lane reverses the whole run.  Both are the same derivative.

Bound: a gradient is a chain of N <= 1,600 steps of some 400 roundings each,
multiplied together in another order by the parts: 1,600 x 400 x 1.1e-16 =
7e-11 of the largest component, times the growth of the parts' unit vectors
against the actual gradient (an omega component weighs up to the step count)."""
import ctypes as C

import numpy as np
import pytest

from paper_0908_3889_amd import population as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
RTOL = 1e-9


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import _lib
    _lib.load()
    yield


def _one_lane(api, _lib, m, omega_f, rec, gy, gt, order=None):
    """pn_integrate_adjoint with a workspace of one segment per inspiral."""
    n, K = int(rec["status"].shape[0]), rec["ckpt_every"]
    nbytes = n * K * 11 * 8
    ws = torch.empty(nbytes // 8, dtype=torch.float64, device="cuda")
    g = {k: torch.empty((c, n) if c > 1 else (n,), dtype=torch.float64, device="cuda")
         for k, c in (("m", 2), ("S0", 6), ("L0", 3), ("omega0", 1))}
    o = api.make_opts()
    p = lambda t: C.c_void_p(t.data_ptr()) if t is not None else None
    rc = _lib.load().pn_integrate_adjoint(n, n, p(m), omega_f, C.byref(o), p(rec["tape"]), rec["cap_steps"], K,
                                          p(rec["status"]), p(gy), p(gt), p(g["m"]), p(g["S0"]), p(g["L0"]),
                                          p(g["omega0"]), p(ws), nbytes, p(order), None)
    _lib.check(rc, "pn_integrate_adjoint")
    torch.cuda.synchronize()
    return g


@pytest.mark.parametrize("workload", ["adjoint_64k", "batching_4M"])
@pytest.mark.parametrize("n,K", [(1, 16), (4, 1), (5, 3), (65, 64), (256, 256), (300, 4096), (1000, 16), (2600, 64),
                                 (5120, 16)])
def test_parts_equal_the_whole_run(workload, n, K):
    from paper_0908_3889_amd import _lib, api
    pop = P.generate(workload, n)
    d = api.to_device(pop)
    rec = api.pn_integrate_record(d["m"], d["S"], d["L"], d["omega0"], pop["omega_f"], pop["tol"], cap_steps=2048,
                                  ckpt_every=K)
    rng = np.random.default_rng(n + K)
    gy = torch.from_numpy(rng.normal(size=(10, n))).cuda()
    for gt in (None, torch.from_numpy(rng.normal(size=n) * 1e-4).cuda()):
        a = api.pn_integrate_adjoint(d["m"], pop["omega_f"], rec, gy, gt)
        b = _one_lane(api, _lib, d["m"], pop["omega_f"], rec, gy, gt)
        for k in a:
            x, y = (v.cpu().numpy().reshape(-1, n) for v in (a[k], b[k]))
            assert np.isfinite(y).all()
            assert (np.abs(x - y) <= RTOL * np.abs(y).max(0)).all(), k


def test_outcomes_order_and_short_runs():
    """Runs of fewer steps than there are parts, of omega-steps alone, failures,
    done at start, a hand-out order with entries that are no index."""
    from paper_0908_3889_amd import _lib, api
    n, K = 40, 2
    pop = P.generate("adjoint_64k", n)
    wf = pop["omega_f"]
    pop["omega0"][:6] = wf * (1.0 - np.array([1e-12, 1e-6, 1e-3, 1e-2, 5e-2, 0.2]))
    pop["omega0"][7] = wf
    pop["m"][0, 9] = -1.0
    d = api.to_device(pop)
    rec = api.pn_integrate_record(d["m"], d["S"], d["L"], d["omega0"], wf, pop["tol"], cap_steps=512, ckpt_every=K)
    assert int(rec["steps"][0].min()) <= 1
    gy = torch.from_numpy(np.random.default_rng(1).normal(size=(10, n))).cuda()
    order = torch.from_numpy(np.random.default_rng(2).permutation(n).astype(np.int32)).cuda()
    a = api.pn_integrate_adjoint(d["m"], wf, rec, gy, order=order)
    b = _one_lane(api, _lib, d["m"], wf, rec, gy, None)
    for k in a:
        x, y = (v.cpu().numpy().reshape(-1, n) for v in (a[k], b[k]))
        np.testing.assert_array_equal(np.isnan(x), np.isnan(y))
        ok = ~np.isnan(y).any(0)
        assert (np.abs(x - y)[:, ok] <= RTOL * np.abs(y[:, ok]).max(0)).all(), k
    order[3], order[11] = -1, n
    c = api.pn_integrate_adjoint(d["m"], wf, rec, gy, order=order)
    kept = np.delete(np.random.default_rng(2).permutation(n), [3, 11])
    for k in a:
        np.testing.assert_array_equal(a[k].cpu().numpy()[..., kept], c[k].cpu().numpy()[..., kept])
