"""The kernel that bench.py says ran, against the library's choice."""
import re

import pytest

import bench
from paper_0908_3889_amd import build

CASES = [dict(n=1), dict(n=1024), dict(n=16384), dict(n=16385), dict(n=65536), dict(n=65537), dict(n=70001, phase=True),
         dict(n=1024, phase=True), dict(n=1024, precision="fp32split"), dict(n=70001, precision="fp32split"),
         dict(n=70001, precision="fp32", phase=True), dict(n=1024, waves_per_simd=2),
         dict(n=70001, waves_per_simd=2, block=128), dict(n=70001, schedule="static", block=64),
         dict(n=70001, order=True, packed=True), dict(n=70001, order=True), dict(n=2097152), dict(n=2097153)]


def _launched(c, cus=256):
    return bench.launched_kernel(c["n"], cus, **{"precision": "fp64", **{k: v for k, v in c.items() if k != "n"}})


def test_names_and_blocks():
    assert _launched(dict(n=16384)) == ("integrate_quad_f64", 256)
    assert _launched(dict(n=1024, phase=True)) == ("integrate_quad_f64_phase", 256)
    assert _launched(dict(n=16385)) == ("integrate_persistent_f64", 256)
    assert _launched(dict(n=1 << 20, order=True, packed=True)) == ("integrate_list_f64", 512)
    assert _launched(dict(n=1 << 20, precision="fp32")) == ("integrate_list_f32x", 768)
    assert _launched(dict(n=1 << 22)) == ("integrate_persistent_f64", 256)
    assert _launched(dict(n=65536), cus=128) == ("integrate_list_f64", 512)


@pytest.mark.parametrize("case", CASES)
def test_resources_are_found(case):
    if not build.resource_usage():
        pytest.skip("library not built (no resource report)")
    r = bench.kernel_resources(*_launched(case))
    assert r and r["VGPRs"] > 100


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_the_library_runs_it(case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import api
    from paper_0908_3889_amd import population as P
    n, phase = case["n"], case.get("phase", False)
    pop = P.generate("adjoint_64k", 64)
    d = api.to_device(pop)
    m, S, L, w = (d[k].repeat(*([1] * (d[k].dim() - 1)), n // 64 + 1)[..., :n].contiguous() for k in ("m", "S", "L", "omega0"))
    w.fill_(0.049)                                     # a few steps
    a = (m, S, L, w, 0.05, 1e-6)
    kw = {k: v for k, v in case.items() if k not in ("n", "phase", "order", "packed")}
    if case.get("order"):
        packed = api.packed_inputs(n)
        kw["order"] = api.pn_cost_order(*a[:5], packed=packed)
        kw["packed"] = packed if case.get("packed") else None
    call = api.pn_integrate_phase if phase else api.pn_integrate
    call(*a, api.make_opts(**kw))
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call(*a, api.make_opts(**kw))
        torch.cuda.synchronize()
    ran = sorted((e.device_time_total, e.key) for e in prof.key_averages() if "integrate_" in e.key)
    kernel, block = _launched(case, torch.cuda.get_device_properties(0).multi_processor_count)
    base = kernel.removesuffix("_phase")
    name = ran[-1][1]                                  # a grid that finds none left runs behind ordered lists
    assert len(ran) == (2 if case.get("packed") else 1), ran
    assert re.search(base + r"(_phase)?<" + str(block), name), (ran, kernel, block)
    if base.split("_")[1] in ("list", "quad"):
        assert (", true>" in name or "true>" in name) == phase, name
    else:
        assert ("_phase<" in name or "true>" in name) == phase, name
