"""The workloads this library is timed on: the softened all-pairs sum, its
vector-Jacobian product, leap-frog integration with its gradient, and
ensembles of independent systems, each through the Python entry points.

``listed()`` names the fixed workloads and ``draw(rng)`` gives others of the
same ranges.  ``prepare`` makes what a program holds before the call (the
particle set, in device memory), ``run`` is one pass, ``work`` the bytes and
operations one pass cannot do without, and ``exact`` the same results in
float64 from plain torch.
"""

import math
import random

import numpy as np
import torch

from paper_0904_3659_amd import leapfrog as lf
from paper_0904_3659_amd import nbody as nb

DEVICE = "cuda"

# Operations of one unordered pair that serves both particles: 3 subtractions,
# 3 FMAs for the squared distance, one reciprocal square root, r^3, one mass
# product and 3 FMAs per side, and one FMA per side for the potential.
FORCE_FLOPS, POTENTIAL_FLOPS = 26, 4
# The same count for the vector-Jacobian product, without and with weights on
# the potential.
VJP_FLOPS, VJP_POTENTIAL_FLOPS = 58, 8

# Above this many bodies the float64 sums take more than some twenty seconds.
EXACT_MAX_N = 400_000


def listed():
    return [
        # One evaluation of a small cluster, the call whose time is the
        # launch: the 1,024-body Plummer sphere of the latency benchmark.
        {"name": "forces_1024", "kind": "forces", "n": 1024, "shape": "plummer", "mass": "equal",
         "eps2": 1e-4, "potential": True},
        # A ragged mid-size system with a mass spectrum (the size the smoke
        # check takes: no multiple of a wave, tile or block).
        {"name": "forces_6001", "kind": "forces", "n": 6001, "shape": "plummer",
         "mass": "lognormal", "eps2": 1e-4, "potential": True},
        # Accelerations only, as an integrator asks for them.
        {"name": "forces_16384_a", "kind": "forces", "n": 16384, "shape": "plummer",
         "mass": "lognormal", "eps2": 1e-4, "potential": False},
        # The ordinary single-GPU evaluation: 65,536 equal masses, a and p.
        {"name": "forces_65536", "kind": "forces", "n": 65536, "shape": "plummer", "mass": "equal",
         "eps2": 1e-4, "potential": True},
        # The largest evaluation of the benchmark, 2^20 bodies with a mass
        # spectrum and a small softening.
        {"name": "forces_1048576", "kind": "forces", "n": 1 << 20, "shape": "plummer",
         "mass": "lognormal", "eps2": 1e-6, "potential": True},
        # Gradient of a loss on (a, p) of a small system, bound by launches.
        {"name": "vjp_1024", "kind": "vjp", "n": 1024, "shape": "plummer", "mass": "lognormal",
         "eps2": 1e-4, "weights_p": True},
        # The adjoint benchmark: 16,384 bodies, weights on a and p.
        {"name": "vjp_16384", "kind": "vjp", "n": 16384, "shape": "plummer", "mass": "lognormal",
         "eps2": 1e-4, "weights_p": True},
        # A large ragged gradient with a loss on the accelerations alone.
        {"name": "vjp_50021_a", "kind": "vjp", "n": 50021, "shape": "cube", "mass": "equal",
         "eps2": 1e-4, "weights_p": False},
        # A short integration of a small cluster: many short launches.
        {"name": "steps_2000", "kind": "steps", "n": 2000, "shape": "plummer", "mass": "equal",
         "eps2": 1e-4, "dt": 0.001, "steps": 64},
        # The paper's run of 100 steps on a 10,000-body galaxy set, with its
        # time step and softening.
        {"name": "steps_10000", "kind": "steps", "n": 10000, "shape": "plummer", "mass": "equal",
         "eps2": 0.01, "dt": 0.015625, "steps": 100},
        # The gradient of a 64-step integration with a checkpoint every 8.
        {"name": "gradient_16384", "kind": "gradient", "n": 16384, "shape": "plummer",
         "mass": "lognormal", "eps2": 1e-4, "dt": 0.001, "steps": 64, "every": 8},
        # 4,096 independent systems of 8 to 2,048 bodies in one call.
        {"name": "ensemble_4096", "kind": "ensemble", "systems": 4096, "least": 8, "most": 2048,
         "layout": 5, "eps2": 1e-4},
    ]


def _spread(rng: random.Random, lo: int, hi: int) -> int:
    """An integer of [lo, hi], uniform over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    kind = rng.choices(("forces", "vjp", "steps", "gradient", "ensemble"), (5, 4, 2, 1, 2))[0]
    case = {"kind": kind, "eps2": rng.choice((1e-6, 1e-4, 1e-2))}
    if kind == "ensemble":
        case |= {"systems": _spread(rng, 16, 4096), "least": rng.choice((1, 8, 100)),
                 "most": _spread(rng, 128, 2048), "layout": rng.randrange(1 << 20)}
        return case
    case |= {"shape": rng.choice(("plummer", "plummer", "cube")),
             "mass": rng.choice(("equal", "lognormal"))}
    if kind == "forces":
        case |= {"n": _spread(rng, 64, 1 << 20), "potential": rng.random() < 0.6}
    elif kind == "vjp":
        case |= {"n": _spread(rng, 64, 1 << 18), "weights_p": rng.random() < 0.5}
    elif kind == "steps":
        case |= {"n": _spread(rng, 256, 100_000), "dt": 0.001, "steps": rng.randint(8, 64)}
    else:
        every = rng.choice((4, 8))
        case |= {"n": _spread(rng, 2100, 20_000), "dt": 0.001,
                 "steps": every * rng.randint(2, 6) + rng.randint(0, 3), "every": every}
    if kind in ("steps", "gradient"):  # no orbit of a close pair shorter than some time steps
        case["eps2"] = rng.choice((1e-4, 1e-2)) if case["shape"] == "plummer" else 1e-2
    return case


# ------------------------------------------------------------------- inputs

def _directions(g, n):
    z = torch.rand(n, generator=g, device=DEVICE, dtype=torch.float64) * 2 - 1
    phi = torch.rand(n, generator=g, device=DEVICE, dtype=torch.float64) * (2 * math.pi)
    rho = (1 - z * z).clamp_min(0).sqrt()
    return torch.stack([rho * phi.cos(), rho * phi.sin(), z], dim=1)


def _positions(g, n, shape):
    if shape == "cube":
        return torch.rand((n, 3), generator=g, device=DEVICE)
    # Plummer sphere of scale radius 1, cut at radius 10, by its inverse CDF
    most = (100.0 / 101.0) ** 1.5
    u = torch.rand(n, generator=g, device=DEVICE, dtype=torch.float64).clamp_min(1e-12) * most
    r = (u.pow(-2.0 / 3.0) - 1).rsqrt().clamp_max(10.0)
    return (r[:, None] * _directions(g, n)).float()


def _masses(g, n, mass):
    if mass == "equal":
        return torch.full((n,), 1.0 / n, device=DEVICE)
    m = torch.randn(n, generator=g, device=DEVICE, dtype=torch.float64).exp()
    return (m / m.sum()).float()


def _velocities(g, x, shape):
    n = x.shape[0]
    if shape == "cube":
        return torch.rand((n, 3), generator=g, device=DEVICE) * 0.2 - 0.1
    # isotropic, with the local velocity dispersion of the sphere
    sigma = (1 + x.double().square().sum(1)).pow(-0.25) / math.sqrt(6)
    v = torch.randn((n, 3), generator=g, device=DEVICE, dtype=torch.float64)
    return (sigma[:, None] * v).float()


def _sizes(case):
    rng = np.random.default_rng(case["layout"])
    return rng.integers(case["least"], case["most"] + 1, case["systems"])


def _inputs(case, seed):
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    s = {}
    if case["kind"] == "ensemble":
        sizes = _sizes(case)
        offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        s["offsets"] = offsets
        s["x"] = _positions(g, int(offsets[-1]), "plummer")
        per_body = np.repeat(1.0 / sizes, sizes).astype(np.float32)
        s["m"] = torch.from_numpy(per_body).to(DEVICE)
        return s
    n = case["n"]
    s["x"] = _positions(g, n, case["shape"])
    s["m"] = _masses(g, n, case["mass"])
    if case["kind"] in ("steps", "gradient"):
        s["v"] = _velocities(g, s["x"], case["shape"])
    if case["kind"] in ("vjp", "gradient"):
        s["w"] = torch.randn((n, 3), generator=g, device=DEVICE)
    if case["kind"] == "vjp":
        s["wp"] = torch.randn(n, generator=g, device=DEVICE) if case["weights_p"] else None
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "gradient":
        for k in ("x", "v", "m"):
            s[k].requires_grad_(True)
    s["case"] = case
    return s


# --------------------------------------------------------------------- pass

def run(s):
    case = s["case"]
    kind, eps2 = case["kind"], case["eps2"]
    if kind == "forces":
        a, p = nb.forces(s["x"], s["m"], eps2, potential=case["potential"])
        return (a, p) if case["potential"] else (a,)
    if kind == "vjp":
        return nb.forces_backward(s["x"], s["m"], eps2, s["w"], s["wp"])
    if kind == "steps":
        x, v, _ = lf.integrate(s["x"], s["v"], s["m"], eps2, case["dt"], case["steps"])
        return x, v
    if kind == "gradient":
        x, v = lf.leapfrog(s["x"], s["v"], s["m"], eps2, case["dt"], case["steps"],
                           checkpoint_every=case["every"])
        gx, gv, gm = torch.autograd.grad(x, (s["x"], s["v"], s["m"]), s["w"])
        return x.detach(), v.detach(), gx, gv, gm
    return nb.forces_batched(s["x"], s["m"], s["offsets"], eps2)


def work(case):
    kind = case["kind"]
    if kind == "ensemble":
        sizes = _sizes(case).astype(np.float64)
        return {"bytes": 32.0 * float(sizes.sum()),
                "flops": (FORCE_FLOPS + POTENTIAL_FLOPS) * float((sizes * (sizes - 1)).sum()) / 2}
    n = float(case["n"])
    pairs = n * (n - 1) / 2
    if kind == "forces":
        p = case["potential"]
        return {"bytes": (32 if p else 28) * n,
                "flops": (FORCE_FLOPS + (POTENTIAL_FLOPS if p else 0)) * pairs}
    if kind == "vjp":
        p = case["weights_p"]
        return {"bytes": (48 if p else 44) * n,
                "flops": (VJP_FLOPS + (VJP_POTENTIAL_FLOPS if p else 0)) * pairs}
    steps = case["steps"]
    if kind == "steps":
        return {"bytes": 52 * n, "flops": (steps + 1) * FORCE_FLOPS * pairs}
    return {"bytes": 92 * n, "flops": ((steps + 1) * FORCE_FLOPS + steps * VJP_FLOPS) * pairs}


# ------------------------------------------------------------- in 64 bits

def _pairs64(x, eps2, lo, hi):
    """(dx, dy, dz, r) of rows lo..hi against every body; r = 0 on i == j."""
    d = [x[lo:hi, c, None] - x[None, :, c] for c in range(3)]
    s = d[0].square()
    s.addcmul_(d[1], d[1]).addcmul_(d[2], d[2]).add_(eps2)
    rows = torch.arange(hi - lo, device=x.device)
    s[rows, rows + lo] = math.inf
    return d, s.rsqrt_()


def _chunks(n):
    rows = max(1, (1 << 25) // n)
    return ((lo, min(n, lo + rows)) for lo in range(0, n, rows))


def _forces64(x, m, eps2, potential=True):
    n = x.shape[0]
    a, p = torch.empty_like(x), torch.empty_like(m) if potential else None
    for lo, hi in _chunks(n):
        d, r = _pairs64(x, eps2, lo, hi)
        if potential:
            p[lo:hi] = torch.mv(r, m)
        f = r.pow(3)
        for c in range(3):
            a[lo:hi, c] = torch.mv(d[c].mul_(f), m)
    return a, p


def _vjp64(x, m, eps2, w, v=None):
    n = x.shape[0]
    gx, gm = torch.empty_like(x), torch.empty_like(m)
    for lo, hi in _chunks(n):
        d, r = _pairs64(x, eps2, lo, hi)
        wk, mk = w[lo:hi], m[lo:hi]
        r3 = r.pow(3)
        wkd = sum(wk[:, c, None] * d[c] for c in range(3))
        wjd = sum(w[None, :, c] * d[c] for c in range(3))
        gm[lo:hi] = -(r3 * wjd).sum(1)
        cd = m[None, :] * wkd - mk[:, None] * wjd
        u = 3 * r.square() * cd
        if v is not None:
            gm[lo:hi] += torch.mv(r, v)
            u += m[None, :] * v[lo:hi, None] + mk[:, None] * v[None, :]
        u *= r3
        A = torch.mv(r3, m)
        for c in range(3):
            B = torch.mv(r3, w[:, c].contiguous())
            gx[lo:hi, c] = wk[:, c] * A - mk * B - (u * d[c]).sum(1)
    return gx, gm


def exact(case, seed):
    kind, eps2 = case["kind"], case["eps2"]
    if case.get("n", 0) > EXACT_MAX_N:
        return None
    s = _inputs(case, seed)
    if kind == "ensemble":
        x, m, o = s["x"].double(), s["m"].double(), s["offsets"].tolist()
        parts = [_forces64(x[lo:hi], m[lo:hi], eps2) for lo, hi in zip(o, o[1:])]
        return torch.cat([a for a, _ in parts]), torch.cat([p for _, p in parts])
    x, m = s["x"].double(), s["m"].double()
    if kind == "forces":
        a, p = _forces64(x, m, eps2, case["potential"])
        return (a, p) if case["potential"] else (a,)
    if kind == "vjp":
        return _vjp64(x, m, eps2, s["w"].double(), None if s["wp"] is None else s["wp"].double())
    dt, steps, n = case["dt"], case["steps"], case["n"]
    evaluations = steps * (4 if kind == "gradient" else 1)
    if evaluations * float(n) ** 2 > 1.5e11:
        return None
    # kick, drift, kick; the physical acceleration is -a
    v = s["v"].double()
    a = _forces64(x, m, eps2, False)[0]
    seen = [x]
    for _ in range(steps):
        v = v - 0.5 * dt * a
        x = x + dt * v
        seen.append(x)
        a = _forces64(x, m, eps2, False)[0]
        v = v - 0.5 * dt * a
    if kind == "steps":
        return x, v
    # the loss is on the final positions: the last kick has no weight
    lx, lv, lm = s["w"].double(), torch.zeros_like(x), torch.zeros_like(m)
    for t in range(steps, 0, -1):
        lv = lv + dt * lx
        gx, gm = _vjp64(seen[t - 1], m, eps2, lv)
        c = -dt if t > 1 else -0.5 * dt
        lx, lm = lx + c * gx, lm + c * gm
    return x, v, lx, lv, lm
