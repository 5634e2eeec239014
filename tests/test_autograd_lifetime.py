"""PNIntegrate's tape lives as long as its outputs, and no longer (CPU: the two
library calls replaced by stand-ins of the same shapes)."""
import gc
import weakref

import pytest

torch = pytest.importorskip("torch")


def _stand_ins(monkeypatch):
    from paper_0908_3889_amd import api
    tapes = []

    def record(m, S0, L0, omega0, omega_f, tol, *, cap_steps, ckpt_every):
        n = omega0.shape[0]
        tape = torch.ones(n, 7, dtype=torch.float64)
        tapes.append(weakref.ref(tape))
        return {"y": torch.cat([omega0[None], S0, L0]).clone(), "t": torch.zeros(n, dtype=torch.float64),
                "status": torch.zeros(n, dtype=torch.int32), "steps": torch.ones((3, n), dtype=torch.int32),
                "tape": tape, "cap_steps": cap_steps, "ckpt_every": ckpt_every}

    def adjoint(m, omega_f, rec, gy, gt, order=None):
        assert rec["tape"].shape[0] == m.shape[1] and rec["cap_steps"] == 32 and rec["ckpt_every"] == 8
        assert (rec["status"] == 0).all() and order.dtype == torch.int32
        return {"m": torch.zeros_like(m), "S0": 2.0 * gy[1:7], "L0": gy[7:10], "omega0": gy[0]}

    monkeypatch.setattr(api, "pn_integrate_record", record)
    monkeypatch.setattr(api, "pn_integrate_adjoint", adjoint)
    n = 3
    args = (torch.ones(2, n, dtype=torch.float64), torch.ones(6, n, dtype=torch.float64, requires_grad=True),
            torch.ones(3, n, dtype=torch.float64), torch.ones(n, dtype=torch.float64))
    return lambda: api.PNIntegrate.apply(*args, 0.05, 1e-8, 8, 32), args[1], tapes


@pytest.fixture()
def no_collector():
    gc.collect()
    gc.disable()
    yield
    gc.enable()


def test_the_tape_goes_with_the_outputs(monkeypatch, no_collector):
    apply, _, tapes = _stand_ins(monkeypatch)
    out = apply()
    assert tapes[0]() is not None
    del out
    assert tapes[0]() is None


def test_the_tape_goes_with_the_backward_pass(monkeypatch, no_collector):
    apply, S0, tapes = _stand_ins(monkeypatch)
    y, t, status, steps = apply()
    y[1:4].sum().backward()
    assert tapes[0]() is None
    want = torch.zeros_like(S0)
    want[:3] = 2.0
    assert torch.equal(S0.grad, want)


def test_a_graph_kept_for_a_second_pass(monkeypatch, no_collector):
    apply, S0, tapes = _stand_ins(monkeypatch)
    y, _, _, _ = apply()
    loss = y[1].sum()
    loss.backward(retain_graph=True)
    loss.backward()
    assert float(S0.grad[0, 0]) == 4.0
    with pytest.raises(RuntimeError):
        loss.backward()


def test_saved_tensor_hooks_see_the_tape(monkeypatch):
    apply, S0, _ = _stand_ins(monkeypatch)
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda x: (seen.append(tuple(x.shape)), x.clone())[1], lambda x: x):
        y, _, _, _ = apply()
    assert (3, 7) in seen
    y[4].sum().backward()
    assert float(S0.grad[3, 0]) == 2.0
