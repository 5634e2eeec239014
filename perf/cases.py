"""The workloads this framework's speed is judged on.

Each case is one pass of a program that uses the public entry points of
``paper_0908_3889_amd.api``: batches of inspirals integrated from omega0 to
omega_f (small batches, where the longest inspiral's chain of steps is the time;
the 1M population; a population with a wide spread of lengths; single precision;
the orbital phase), one point of a parameter study, gradients of a loss on the
final states, the statistics of the scalar products of the spins and the orbital
angular momentum, initial data drawn on the GPU, and the streamed
Kolmogorov-Smirnov run.

``exact`` is the same mathematics in plain torch or numpy in 64 bits: Eqs. (1)-(4)
with the adaptive Dormand-Prince method written on whole arrays, its gradients by
torch's own differentiation with the accepted step sizes held fixed, the
statistics from their definitions, and the Philox4x64-10 draws.
"""
import math

import numpy as np
import torch

from paper_0908_3889_amd import api

# The populations: mass ratio q = m1/m2 uniform, Kerr parameters uniform, spin
# directions isotropic, omega0 log-uniform (fixed where the ends are equal), M = 1.
POPULATIONS = {
    # equal masses at maximal spin, tight tolerance: the smallest batch
    "equal_mass": dict(q=(1.0, 1.0), chi=(1.0, 1.0), omega0=(0.01, 0.01), omega_f=0.05, tol=1e-10),
    # the paper's science setting (equal masses, maximal spin, long inspirals)
    "study": dict(q=(1.0, 1.0), chi=(1.0, 1.0), omega0=(0.00395, 0.00395), omega_f=0.05, tol=5e-7),
    # the default population of the benchmark
    "q1to4": dict(q=(1.0, 4.0), chi=(0.0, 1.0), omega0=(0.005, 0.005), omega_f=0.05, tol=1e-8),
    # a wide spread of lengths (about 20x between the shortest and the longest)
    "wide": dict(q=(1.0, 10.0), chi=(0.0, 1.0), omega0=(0.002, 0.01), omega_f=0.05, tol=1e-8),
    # the population that gradients are taken on
    "gradient": dict(q=(1.0, 4.0), chi=(0.5, 1.0), omega0=(0.01, 0.01), omega_f=0.05, tol=1e-8),
}


def listed():
    return [
        # A thousand inspirals at tight tolerance: a quick look at one setting, or a
        # chunk of a parameter scan.  The chip is nearly empty; latency is the time.
        dict(name="integrate_1k", kind="integrate", population="equal_mass", n=1024, precision="fp64",
             ordered=False, phase=False),
        # One point of a parameter study: integrate a population, then Pearson's r of the
        # initial against the final scalar products.
        dict(name="study_16k", kind="study", population="study", n=16384),
        # Waveform-style outputs: the orbital phase alongside, a batch of odd size.
        dict(name="phase_100k", kind="integrate", population="q1to4", n=100003, precision="fp64", ordered=False,
             phase=True),
        # The benchmark's population: longest-first order and packed records for new
        # inputs, then the integration.
        dict(name="integrate_1m", kind="integrate", population="q1to4", n=1 << 20, precision="fp64", ordered=True,
             phase=False),
        # Inspirals of very different lengths sharing the chip, an odd size.
        dict(name="integrate_wide_500k", kind="integrate", population="wide", n=500009, precision="fp64",
             ordered=True, phase=False),
        # The paper's single precision with a few computations in double.
        dict(name="fp32split_1m", kind="integrate", population="q1to4", n=1 << 20, precision="fp32split",
             ordered=True, phase=False),
        # Gradients of a loss on the final states, forward and backward: a small batch,
        # as an optimiser over a few hundred binaries calls it ...
        dict(name="gradient_1k", kind="gradient", population="gradient", n=1000, every=16),
        # ... and a batch that fills the chip.
        dict(name="gradient_64k", kind="gradient", population="gradient", n=65536, every=64),
        # The statistics stage after a small run (launches count) and after the 1M run.
        dict(name="statistics_4k", kind="statistics", n=4099, nbins=20, nbins2d=79, ngrid=201),
        dict(name="statistics_1m", kind="statistics", n=1 << 20, nbins=20, nbins2d=79, ngrid=201),
        # Initial data for one chunk of a streamed run.
        dict(name="generate_4m", kind="generate", n=1 << 22, first=1 << 33),
        # The streamed Kolmogorov-Smirnov run: generate, integrate, keep the final
        # S1.S2, test the whole sample; the last chunk is ragged.
        dict(name="ks_run_1m", kind="ks_run", total=1200007, chunk=1 << 19, nbins=100),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["integrate", "integrate", "integrate", "study", "gradient", "statistics", "generate", "ks_run"])
    if kind == "integrate":
        precision = rng.choice(["fp64", "fp64", "fp32split", "fp32"])
        n = _log_int(rng, 64, 1 << 20)
        population = rng.choice(["equal_mass", "study", "q1to4", "wide", "gradient"])
        if population == "wide":
            n = min(n, 500009)
        return dict(kind=kind, population=population, n=n, precision=precision, ordered=n >= 1 << 17,
                    phase=rng.random() < 0.25)
    if kind == "study":
        return dict(kind=kind, population="study", n=_log_int(rng, 1024, 65536))
    if kind == "gradient":
        return dict(kind=kind, population="gradient", n=_log_int(rng, 64, 65536), every=rng.choice([16, 64, 256]))
    if kind == "statistics":
        return dict(kind=kind, n=_log_int(rng, 1000, 1 << 20), nbins=rng.choice([20, 100, 37]),
                    nbins2d=rng.choice([79, 64, 25]), ngrid=rng.choice([201, 101, 400, 257]))
    if kind == "generate":
        return dict(kind=kind, n=_log_int(rng, 1024, 1 << 22), first=rng.randrange(1 << 40))
    return dict(kind=kind, total=_log_int(rng, 40000, 1200007), chunk=rng.choice([1 << 16, 1 << 18, 1 << 19]),
                nbins=rng.choice([20, 100]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _directions(g, n):
    v = torch.randn(3, n, generator=g, device="cuda", dtype=torch.float64)
    return v / v.norm(dim=0)


def _population(case, seed):
    """Masses, spins, L_hat = z and omega0 of the case's population, structure of arrays."""
    p, n, g = POPULATIONS[case["population"]], case["n"], _generator(seed)
    q = _uniform(g, *p["q"], n)
    m = torch.stack([q / (1.0 + q), 1.0 / (1.0 + q)])
    chi1, chi2 = _uniform(g, *p["chi"], n), _uniform(g, *p["chi"], n)
    S = torch.cat([chi1 * m[0] ** 2 * _directions(g, n), chi2 * m[1] ** 2 * _directions(g, n)])
    L = torch.zeros(3, n, device="cuda", dtype=torch.float64)
    L[2] = 1.0
    lo, hi = p["omega0"]
    omega0 = torch.full((n,), lo, device="cuda", dtype=torch.float64)
    if hi > lo:
        omega0 = torch.exp(_uniform(g, math.log(lo), math.log(hi), n))
    return {"m": m, "S": S, "L": L, "omega0": omega0}


def _scalar_products(case, seed):
    """Initial and final scalar products of S1, S2, L as a run gives them: of isotropic
    unit vectors, and of the same vectors after a spread of rotations."""
    n, g = case["n"], _generator(seed)

    def dots(a, b, c):
        return torch.stack([(a * b).sum(0), (a * c).sum(0), (b * c).sum(0)])

    v = [_directions(g, n) for _ in range(3)]
    w = []
    for a, s in zip(v, (0.25, 0.4, 0.1)):
        b = a + s * torch.randn(3, n, generator=g, device="cuda", dtype=torch.float64)
        w.append(b / b.norm(dim=0))
    return dots(*v).clamp(-1.0, 1.0).contiguous(), dots(*w).clamp(-1.0, 1.0).contiguous()


def _spec(case, seed):
    """The distributions of the GPU's draw: the benchmark's for a population, the paper's
    setting at Kerr parameter 0.7 for the K-S run."""
    if case["kind"] == "generate":
        return dict(q=(1.0, 4.0), chi1=(0.0, 1.0), chi2=(0.0, 1.0), omega0=(0.005, 0.01), seed=seed)
    return dict(q=(1.0, 1.0), chi1=(0.7, 0.7), chi2=(0.7, 0.7), omega0=(0.00395, 0.00395), seed=seed)


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind in ("integrate", "study", "gradient"):
        p, n = POPULATIONS[case["population"]], case["n"]
        state.update(_population(case, seed), omega_f=p["omega_f"], tol=p["tol"])
        if kind == "integrate":
            state["out"] = api.alloc_outputs(n)
            if case["phase"]:
                state["out"]["phase"] = torch.empty(n, device="cuda", dtype=torch.float64)
            order = packed = None
            if case["ordered"]:
                order = torch.empty(n, device="cuda", dtype=torch.int32)
                packed = api.packed_inputs(n)
                state.update(order=order, packed=packed, workspace=api.cost_order_workspace(n))
            state["opts"] = api.make_opts(precision=case["precision"], order=order, packed=packed)
    elif kind == "statistics":
        state["initial"], state["final"] = _scalar_products(case, seed)
    elif kind == "generate":
        state["spec"] = api.gen_spec(**_spec(case, seed))
    elif kind == "ks_run":
        state["spec"] = api.gen_spec(**_spec(case, seed))
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "integrate":
        args = (state["m"], state["S"], state["L"], state["omega0"], state["omega_f"])
        if case["ordered"]:
            api.pn_cost_order(*args, out=state["order"], workspace=state["workspace"], packed=state["packed"])
        call = api.pn_integrate_phase if case["phase"] else api.pn_integrate
        return call(*args, state["tol"], state["opts"], out=state["out"])
    if kind == "study":
        out = api.pn_integrate(state["m"], state["S"], state["L"], state["omega0"], state["omega_f"], state["tol"])
        out["pearson"] = api.pn_pearson(api.initial_dots(state), out["dots"])
        return out
    if kind == "gradient":
        # the loss sum S1.S2 + sum L_z on the final states: its gradient seeds the reverse sweep,
        # the inspirals in the order of their step counts
        rec = api.pn_integrate_record(state["m"], state["S"], state["L"], state["omega0"], state["omega_f"],
                                      state["tol"], cap_steps=2048, ckpt_every=case["every"])
        y = rec["y"]
        seed = torch.zeros_like(y)
        seed[1:4], seed[4:7], seed[9] = y[4:7], y[1:4], 1.0
        order = torch.argsort(rec["steps"][0], descending=True).to(torch.int32)
        grads = api.pn_integrate_adjoint(state["m"], state["omega_f"], rec, seed, order=order)
        return {"y": y, "t": rec["t"], "status": rec["status"], "steps": rec["steps"], "grads": grads}
    if kind == "statistics":
        return api.statistics(state["initial"], state["final"], case["nbins"], case["nbins2d"], case["ngrid"])
    if kind == "generate":
        return api.pn_generate(case["n"], state["spec"], case["first"])
    p = POPULATIONS["study"]
    return api.ks_run(case["total"], state["spec"], p["omega_f"], p["tol"], case["chunk"], case["nbins"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

RHS_FLOP, STEP_FLOP = 101, 586     # one evaluation of Eqs. (1)-(4); the rest of an attempted step


def _steps(population):
    """Attempted steps of one inspiral: proportional to the precession angle, which grows
    as 1/omega0 - 1/omega_f, and to tol^(-1/5) (means over the populations)."""
    p = POPULATIONS[population]
    lo, hi = p["omega0"]
    inv = 1.0 / lo if hi == lo else (1.0 / lo - 1.0 / hi) / math.log(hi / lo)
    return 20.0 + 1.2 * (inv - 1.0 / p["omega_f"]) * (p["tol"] / 1e-8) ** -0.2


def work(case):
    kind = case["kind"]
    if kind in ("integrate", "study", "gradient"):
        n, steps = case["n"], _steps(case["population"])
        flops = n * steps * (6 * RHS_FLOP + STEP_FLOP)
        nbytes = n * (12 * 8 + 11 * 8 + 4 * 4 + 3 * 8)
        if kind == "gradient":
            # the reverse sweep recomputes the stages of a step and takes one transposed
            # Jacobian product (about twice an evaluation) per stage; step sizes and
            # checkpoints written once and read once
            flops += n * steps * (6 * 3 * RHS_FLOP + 2 * 400)
            nbytes += n * (12 * 8 + 10 * 8 + 2 * 8 * (steps + 10 * steps / case["every"]))
        return {"bytes": nbytes, "flops": flops}
    if kind == "statistics":
        n = case["n"]
        # per value: a bin, a pair of bins, the sums of r, one kernel value per grid point, and a place in the sorted order
        return {"bytes": 2 * 3 * n * 8, "flops": 3.0 * n * (2 * case["ngrid"] + 30)}
    if kind == "generate":
        return {"bytes": case["n"] * 12 * 8, "flops": case["n"] * 60}
    return {"bytes": case["total"] * (12 + 12 + 14 + 2) * 8,
            "flops": case["total"] * _steps("study") * (6 * RHS_FLOP + STEP_FLOP)}


# ---------------------------------------------------------------------------
# the same mathematics in 64 bits
# ---------------------------------------------------------------------------

def _row(m):
    """Everything in Eqs. (1)-(4) that depends on the masses alone."""
    m1, m2 = m[0], m[1]
    M = m1 + m2
    eta = m1 * m2 / M ** 2
    pi = math.pi
    c6 = (16447322263.0 / 139708800.0 - 1712.0 / 105.0 * 0.57721566490153286061 + 16.0 / 3.0 * pi ** 2
          + (-273811877.0 / 1088640.0 + 451.0 / 48.0 * pi ** 2 - 88.0 / 3.0 * (1039.0 / 4620.0)) * eta
          + 541.0 / 896.0 * eta ** 2 - 5605.0 / 2592.0 * eta ** 3 - 856.0 / 105.0 * math.log(16.0))
    return torch.stack([
        M, -(743.0 + 924.0 * eta) / 336.0,
        (113.0 * (m1 / M) ** 2 + 75.0 * eta) / (12.0 * m1 ** 2), (113.0 * (m2 / M) ** 2 + 75.0 * eta) / (12.0 * m2 ** 2),
        34103.0 / 18144.0 + 13661.0 / 2016.0 * eta + 59.0 / 18.0 * eta ** 2, eta / (48.0 * m1 ** 2 * m2 ** 2),
        -(4159.0 + 15876.0 * eta) * pi / 672.0, c6,
        (-4415.0 / 4032.0 + 358675.0 / 6048.0 * eta + 91495.0 / 1512.0 * eta ** 2) * pi,
        96.0 / 5.0 * eta, eta * (4.0 + 3.0 * m2 / m1), eta * (4.0 + 3.0 * m1 / m2), 1.0 / M, 1.0 / (eta * M ** 2)])


def _cross(a, b):
    return torch.linalg.cross(a, b, dim=0)


def _rhs(r, y):
    """dy/dt of Eqs. (1)-(4), y = (omega, S1, S2, L_hat)."""
    w, S1, S2, L = y[0], y[1:4], y[4:7], y[7:10]
    v = r[0] * w
    x = v.abs() ** (1.0 / 3.0) * v.sign()
    x2 = x * x
    LS1, LS2, S12 = (L * S1).sum(0), (L * S2).sum(0), (S1 * S2).sum(0)
    c3 = 4.0 * math.pi - r[2] * LS1 - r[3] * LS2
    c4 = r[4] - r[5] * (247.0 * S12 - 721.0 * LS1 * LS2)
    c6 = r[7] - 1712.0 / 315.0 * v.abs().log()
    B = 1.0 + x2 * (r[1] + x * (c3 + x * (c4 + x * (r[6] + x * (c6 + x * r[8])))))
    dw = r[9] * w * w * x2 * v * B
    p, sv = 0.5 * w, r[12] * w
    dS1 = _cross(p * ((r[10] * x2 - 3.0 * sv * LS2) * L + sv * S2), S1)
    dS2 = _cross(p * ((r[11] * x2 - 3.0 * sv * LS1) * L + sv * S1), S2)
    return torch.cat([dw[None], dS1, dS2, -r[13] * x * (dS1 + dS2)])


def _derivative(r, y, om):
    """The derivative along the step's variable (t, or omega where om) and dt along it."""
    k = _rhs(r, y)
    if om is None:
        return k, torch.ones_like(k[0])
    s = torch.where(om, 1.0 / k[0], torch.ones_like(k[0]))
    return torch.cat([torch.where(om, torch.ones_like(s), k[0])[None], k[1:] * s]), s


# Dormand & Prince (1980)
A = [[1 / 5], [3 / 40, 9 / 40], [44 / 45, -56 / 15, 32 / 9], [19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729],
     [9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656]]
B5 = [35 / 384, 0.0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84]
E5 = [71 / 57600, 0.0, -71 / 16695, 71 / 1920, -17253 / 339200, 22 / 525, -1 / 40]


def _stages(r, y, k1, d1, h, om):
    k, d, w = [k1], [d1], [y[0]]
    for row in A:
        Y = y + h * sum(a * kj for a, kj in zip(row, k))
        kj, dj = _derivative(r, Y, om)
        k.append(kj), d.append(dj), w.append(Y[0])
    ynew = y + h * sum(b * kj for b, kj in zip(B5, k) if b)
    dt = h * sum(b * dj for b, dj in zip(B5, d) if b)
    dphi = h * sum(b * dj * wj for b, dj, wj in zip(B5, d, w) if b)
    return k, ynew, dt, dphi


def _integrate(y0, m, omega_f, tol, tape=None):
    """Adaptive Dormand-Prince from omega0 to omega_f, the last stretch in omega, on the whole
    batch; finished inspirals leave the arrays.  tape: a list that receives each pass's
    (step size, omega-step, last step), whole batch, zero where nothing was accepted."""
    n, dev = y0.shape[1], y0.device
    out = {"y": y0.clone(), "t": torch.zeros(n, device=dev, dtype=torch.float64),
           "phase": torch.zeros(n, device=dev, dtype=torch.float64)}
    idx = torch.arange(n, device=dev)
    r, y = _row(m), y0.clone()
    t, phase = torch.zeros_like(out["t"]), torch.zeros_like(out["t"])
    h = torch.full_like(t, 10.0)
    om = torch.zeros(n, device=dev, dtype=torch.bool)
    rejected = torch.zeros_like(om)
    k1, d1 = _derivative(r, y, None)
    done = torch.zeros_like(om)
    count = 0
    while True:
        remain = omega_f - y[0]
        last = om & (h >= remain)
        hh = torch.where(last, remain, h)
        hh = torch.where(done, torch.zeros_like(hh), hh)
        k, ynew, dt, dphi = _stages(r, y, k1, d1, hh, om)
        k7, d7 = _derivative(r, ynew, om)
        e = hh * (sum(c * kj for c, kj in zip(E5, k) if c) + E5[6] * k7)
        z = ((e / (tol + tol * torch.maximum(y.abs(), ynew.abs()))) ** 2).mean(0)
        ok = (z <= 1.0 + 2.0 ** -52) & ~done
        to_w = ok & ~om & (ynew[0] > omega_f)
        take, rej = ok & ~to_w, ~ok & ~done
        p = 0.9 * z.clamp(2.0 ** -30, 2.0 ** 30) ** -0.1
        p = p.clamp(min=0.2)
        fac = torch.where(rej, p, torch.minimum(p, torch.where(rejected, 1.0, 5.0)))
        if tape is not None:
            tape.append((torch.where(take, hh, torch.zeros_like(hh)), om.clone(), take & last))
        end = take & (last | (~om & (ynew[0] == omega_f)))
        s = torch.where(to_w, 1.0 / k1[0], torch.ones_like(t))
        k1 = torch.cat([torch.where(to_w, torch.ones_like(s), k1[0])[None], k1[1:] * s])
        d1 = torch.where(to_w, s, d1)
        y, k1, d1 = torch.where(take, ynew, y), torch.where(take, k7, k1), torch.where(take, d7, d1)
        y[0] = torch.where(end, torch.full_like(t, omega_f), y[0])
        t, phase = torch.where(take, t + torch.where(om, dt, hh), t), torch.where(take, phase + dphi, phase)
        resize = rej | (take & ~end)
        h = torch.where(to_w, omega_f - y[0], torch.where(resize, hh * fac, h))
        rejected = torch.where(to_w, torch.zeros_like(rejected), torch.where(resize, rej, rejected))
        om, done = om | to_w, done | end
        count += 1
        if count % 16:
            continue
        live = ~done
        left = int(live.sum())
        if tape is not None:
            if left == 0:
                out.update(y=y, t=t, phase=phase)
                return out
            continue
        if left < 0.8 * idx.numel():
            f = idx[done]
            out["y"][:, f], out["t"][f], out["phase"][f] = y[:, done], t[done], phase[done]
            if left == 0:
                return out
            idx, r, y, k1 = idx[live], r[:, live], y[:, live], k1[:, live]
            t, phase, h, d1, om, rejected, done = (a[live] for a in (t, phase, h, d1, om, rejected, done))


def _products(y):
    a, b, c = (v / v.norm(dim=0) for v in (y[1:4], y[4:7], y[7:10]))
    return torch.stack([(a * b).sum(0), (a * c).sum(0), (b * c).sum(0)])


def _pearson(x, y):
    n = x.shape[1]
    mx, my = x.mean(1), y.mean(1)
    dx, dy = x - mx[:, None], y - my[:, None]
    sx, sy = (dx * dx).sum(1), (dy * dy).sum(1)
    return torch.stack([mx, my, (sx / (n - 1)).sqrt(), (sy / (n - 1)).sqrt(), (dx * dy).sum(1) / (sx * sy).sqrt()], 1)


def _kde(x, sigma, ngrid):
    n = x.shape[1]
    h = 1.06 * sigma * n ** -0.2
    grid = -1.0 + torch.arange(ngrid, device=x.device, dtype=torch.float64) * (2.0 / (ngrid - 1))
    out = torch.zeros(x.shape[0], ngrid, device=x.device, dtype=torch.float64)
    for a in range(0, n, 1 << 15):
        u = (grid[None, :, None] - x[:, None, a:a + (1 << 15)]) / h[:, None, None]
        out += torch.exp(-0.5 * u * u).sum(2)
    return out / (n * h[:, None] * math.sqrt(2.0 * math.pi))


def _ks(x, lo=-1.0, hi=1.0):
    n = x.shape[-1]
    F = (x.sort().values - lo) / (hi - lo)
    i = torch.arange(n, device=x.device, dtype=torch.float64)
    d = float(torch.maximum((i + 1) / n - F, F - i / n).max())
    lam = math.sqrt(n) * d
    if lam >= 1.0:
        p = sum((2.0 if k & 1 else -2.0) * math.exp(-2.0 * k * k * lam * lam) for k in range(1, 101))
    else:
        p = 1.0 - math.sqrt(2.0 * math.pi) / lam * sum(
            math.exp(-(2 * k - 1) ** 2 * math.pi ** 2 / (8.0 * lam * lam)) for k in range(1, 101))
    return torch.tensor([d, min(max(p, 0.0), 1.0)], device=x.device, dtype=torch.float64)


def _mulhi(a, b):
    """Upper 64 bits of the 128-bit product (numpy uint64)."""
    lo32, s = np.uint64(0xFFFFFFFF), np.uint64(32)
    a0, a1, b0, b1 = a & lo32, a >> s, b & lo32, b >> s
    mid = a1 * b0 + ((a0 * b0) >> s)
    return a1 * b1 + (mid >> s) + ((a0 * b1 + (mid & lo32)) >> s)


def _philox(counter, block, seed):
    """Philox4x64-10 of (counter, block, 0, 0) under the key (seed, 0)."""
    M0, M1 = np.uint64(0xD2E7470EE14C6C93), np.uint64(0xCA5A826395121157)
    W0, W1 = 0x9E3779B97F4A7C15, 0xBB67AE8584CAA73B
    x = [counter, np.full_like(counter, block), np.zeros_like(counter), np.zeros_like(counter)]
    for i in range(10):
        k0, k1 = (np.uint64((k + i * w) % (1 << 64)) for k, w in ((seed, W0), (0, W1)))
        x = [_mulhi(M1, x[2]) ^ x[1] ^ k0, M1 * x[2], _mulhi(M0, x[0]) ^ x[3] ^ k1, M0 * x[0]]
    return [(v >> np.uint64(11)).astype(np.float64) * 2.0 ** -53 for v in x]


def _sphere(counter, block, seed):
    """Marsaglia's points on the sphere, two attempts a block."""
    out = np.zeros((3, counter.size))
    out[2] = 1.0
    left = np.arange(counter.size)
    for b in range(32):
        u = _philox(counter[left], block + b, seed)
        todo = np.ones(left.size, dtype=bool)
        for u1, u2 in ((u[0], u[1]), (u[2], u[3])):
            a, c = 2.0 * u1 - 1.0, 2.0 * u2 - 1.0
            s = a * a + c * c
            fine = todo & (s < 1.0)
            f = 2.0 * np.sqrt(np.where(fine, 1.0 - s, 0.0))
            out[:, left[fine]] = np.stack([a * f, c * f, 1.0 - 2.0 * s])[:, fine]
            todo &= ~fine
        left = left[todo]
        if left.size == 0:
            break
    return out


def _draws(n, first, spec):
    counter = np.arange(first, first + n, dtype=np.uint64)
    seed = spec["seed"]
    u = _philox(counter, 0, seed)
    q, c1, c2, w = (lo + (hi - lo) * v for (lo, hi), v in
                    zip((spec["q"], spec["chi1"], spec["chi2"], spec["omega0"]), u))
    m1, m2 = q / (1.0 + q), 1.0 / (1.0 + q)
    S = np.concatenate([c1 * m1 ** 2 * _sphere(counter, 1, seed), c2 * m2 ** 2 * _sphere(counter, 33, seed)])
    L = np.zeros((3, n))
    L[2] = 1.0
    return {"m": np.stack([m1, m2]), "S": S, "L": L, "omega0": w}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("integrate", "study", "gradient"):
        p, d = POPULATIONS[case["population"]], _population(case, seed)
        y0 = torch.cat([d["omega0"][None], d["S"], d["L"]])
    if kind in ("integrate", "study"):
        o = _integrate(y0, d["m"], p["omega_f"], p["tol"])
        res = {"y": o["y"], "t": o["t"], "steps": None, "status": None, "dots": _products(o["y"])}
        if kind == "study":
            res["pearson"] = _pearson(_products(y0), res["dots"])
        elif case["phase"]:
            res["phase"] = o["phase"]
        return res
    if kind == "gradient":
        tape = []
        o = _integrate(y0, d["m"], p["omega_f"], p["tol"], tape)
        r = _row(d["m"])

        def step(r, y, h, om, last):
            h = torch.where(last, p["omega_f"] - y[0], h)
            k1, d1 = _derivative(r, y, om)
            return torch.where(h != 0.0, _stages(r, y, k1, d1, h, om)[1], y)

        # the steps forward, then their transposed derivatives one at a time from the last
        states = [y0]
        for h, om, last in tape:
            states.append(step(r, states[-1], h, om, last))
        y = states.pop()
        gy, gr = torch.zeros_like(y), torch.zeros_like(r)
        gy[1:4], gy[4:7], gy[9] = y[4:7], y[1:4], 1.0
        for (h, om, last), yk in zip(reversed(tape), reversed(states)):
            inputs = (r.detach().requires_grad_(True), yk.detach().requires_grad_(True))
            dr, gy = torch.autograd.grad(step(*inputs, h, om, last), inputs, gy)
            gr += dr
        m = d["m"].requires_grad_(True)
        grads = {"m": torch.autograd.grad(_row(m), m, gr)[0], "S0": gy[1:7], "L0": gy[7:10], "omega0": gy[0]}
        return {"y": o["y"], "t": o["t"], "status": None, "steps": None, "grads": grads}
    if kind == "statistics":
        x, y = _scalar_products(case, seed)
        pr = _pearson(x, y)
        return {"hist": None, "hist2d": None, "pearson": pr, "kde": _kde(y, pr[:, 3], case["ngrid"]),
                "ks": torch.stack([_ks(c) for c in y])}
    if kind == "generate":
        return _draws(case["n"], case["first"], _spec(case, seed))
    p = POPULATIONS["study"]
    d = {k: torch.from_numpy(v).cuda() for k, v in _draws(case["total"], 0, _spec(case, seed)).items()}
    o = _integrate(torch.cat([d["omega0"][None], d["S"], d["L"]]), d["m"], p["omega_f"], p["tol"])
    s1s2 = _products(o["y"])[0]
    return {"n": None, "ks": _ks(s1s2), "hist": None, "not_ok": None, "final_s1s2": s1s2}
