"""Gradients of small batches in a launch that leaves SIMDs to other streams: with
waves_per_simd set, one lane reverses each inspiral's whole run, as in a workspace
of one segment per inspiral; and the workspaces between that size and the full one,
whose size is the number of parts."""
import ctypes as C

import numpy as np
import pytest

from paper_0908_3889_amd import population as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

RTOL = 1e-9      # of the largest component: test_gpu_adjoint_parts.py


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import _lib
    _lib.load()
    yield


def _record(n, K):
    from paper_0908_3889_amd import api
    pop = P.generate("adjoint_64k", n)
    d = api.to_device(pop)
    rec = api.pn_integrate_record(d["m"], d["S"], d["L"], d["omega0"], pop["omega_f"], pop["tol"], cap_steps=512,
                                  ckpt_every=K)
    gy = torch.from_numpy(np.random.default_rng(n).normal(size=(10, n))).cuda()
    return d["m"], pop["omega_f"], rec, gy


def _in(words, m, omega_f, rec, gy, guard=4096):
    """pn_integrate_adjoint in a workspace of `words` doubles, with as many known
    values behind it that must stay."""
    from paper_0908_3889_amd import _lib, api
    n = int(rec["status"].shape[0])
    ws = torch.full((words + guard,), 123.25, dtype=torch.float64, device="cuda")
    g = {k: torch.empty((c, n) if c > 1 else (n,), dtype=torch.float64, device="cuda")
         for k, c in (("m", 2), ("S0", 6), ("L0", 3), ("omega0", 1))}
    p = lambda t: C.c_void_p(t.data_ptr())
    rc = _lib.load().pn_integrate_adjoint(n, n, p(m), omega_f, C.byref(api.make_opts()), p(rec["tape"]),
                                          rec["cap_steps"], rec["ckpt_every"], p(rec["status"]), p(gy), None, p(g["m"]),
                                          p(g["S0"]), p(g["L0"]), p(g["omega0"]), p(ws), 8 * words, None, None)
    _lib.check(rc, "pn_integrate_adjoint")
    torch.cuda.synchronize()
    assert (ws[words:] == 123.25).all()
    return g


@pytest.mark.parametrize("n,K", [(1, 16), (300, 64), (3000, 16)])
def test_waves_per_simd_reverses_the_whole_run(n, K):
    from paper_0908_3889_amd import api
    m, omega_f, rec, gy = _record(n, K)
    a = api.pn_integrate_adjoint(m, omega_f, rec, gy, opts=api.make_opts(waves_per_simd=2))
    b = _in(n * K * 11, m, omega_f, rec, gy)
    for k in a:
        assert torch.equal(a[k], b[k]), k


# parts c take c segments of 11 n K doubles, and 24 n (1 + 11 (c - 1)) of what they
# hand on: those sizes, and a double fewer
@pytest.mark.parametrize("n,K", [(5, 3), (130, 16), (1000, 16)])
def test_workspaces_of_two_parts_and_more(n, K):
    from paper_0908_3889_amd import _lib
    args = _record(n, K)
    whole = _in(n * K * 11, *args)
    full = int(_lib.load().pn_adjoint_workspace_bytes(n, K)) // 8
    size = lambda c: c * n * K * 11 + 24 * n * (1 + 11 * (c - 1))
    most = max(c for c in range(1, 17) if size(c) <= full)
    assert most > 1 and size(most) == full
    for c in range(2, most + 1):
        for words in (size(c) - 1, size(c)):
            got = _in(words, *args)
            for k in got:
                x, y = (v.cpu().numpy().reshape(-1, n) for v in (got[k], whole[k]))
                assert (np.abs(x - y) <= RTOL * np.abs(y).max(0)).all(), (c, words, k)
