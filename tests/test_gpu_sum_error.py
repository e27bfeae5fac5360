"""How far the float32 results are from float64: the sums over pairs may not
lose more than the plain form of each kernel does (one tile's pairs to a float32
sum, one partial per tile or chunk, the partials added in float64).

Each bound is the error (2-norm over the rows of two particle sets, relative)
that kernels of that form gave on the same inputs, plus 2%; the present forms
(more rows per lane, several waves to a partial, row groups) have to stay below.
"""

import pytest
import torch

from paper_0904_3659_amd import inputs
from tests.gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu

ROWS = 4096  # rows compared, evenly spaced

# n, masses, positions(, potential weights), error of the plain form (vectors, scalars);
# eps2 = 0.01
FORWARD = [
    (5003, "equal", "cube", (3.783e-08, 3.014e-08)),
    (5003, "lognormal", "plummer", (4.643e-08, 2.997e-08)),
    (10000, "equal", "cube", (3.504e-08, 2.755e-08)),
    (10000, "lognormal", "plummer", (4.013e-08, 2.716e-08)),
    (12001, "equal", "cube", (3.488e-08, 2.737e-08)),
    (12001, "lognormal", "plummer", (3.964e-08, 2.661e-08)),
    (16384, "lognormal", "plummer", (3.809e-08, 2.584e-08)),
    (30000, "lognormal", "plummer", (3.777e-08, 2.706e-08)),
    (50021, "equal", "cube", (3.416e-08, 2.697e-08)),
    (50021, "lognormal", "plummer", (3.707e-08, 2.676e-08)),
    (65536, "lognormal", "plummer", (3.646e-08, 2.573e-08)),
    (262144, "lognormal", "plummer", (3.630e-08, 2.692e-08)),
    (1048576, "lognormal", "plummer", (3.816e-08, 2.979e-08)),
]
ADJOINT = [
    (4501, "equal", "cube", True, (7.794e-08, 1.984e-07)),
    (4501, "lognormal", "cube", False, (8.639e-08, 1.620e-07)),
    (4501, "lognormal", "plummer", True, (1.420e-07, 1.975e-07)),
    (6001, "equal", "cube", True, (7.465e-08, 2.116e-07)),
    (6001, "lognormal", "cube", False, (8.012e-08, 1.838e-07)),
    (6001, "lognormal", "plummer", True, (1.420e-07, 1.972e-07)),
    (8000, "equal", "cube", True, (7.234e-08, 2.239e-07)),
    (8000, "lognormal", "cube", False, (7.198e-08, 1.913e-07)),
    (8000, "lognormal", "plummer", True, (1.283e-07, 1.914e-07)),
    (11000, "equal", "cube", True, (6.975e-08, 2.252e-07)),
    (11000, "lognormal", "cube", False, (6.619e-08, 1.883e-07)),
    (11000, "lognormal", "plummer", True, (1.161e-07, 1.904e-07)),
    (16384, "lognormal", "cube", False, (6.386e-08, 2.144e-07)),
    (16384, "lognormal", "plummer", True, (1.155e-07, 2.750e-07)),
    (30000, "equal", "cube", True, (6.674e-08, 2.249e-07)),
    (50021, "lognormal", "cube", False, (4.992e-08, 1.829e-07)),
    (50021, "lognormal", "plummer", True, (8.171e-08, 2.842e-07)),
    (262144, "lognormal", "plummer", True, (6.459e-08, 2.989e-07)),
]


@pytest.fixture(scope="module")
def nb():
    need_gpu()
    from paper_0904_3659_amd import nbody
    return nbody


def _system(n, mass, shape, key, dev):
    x = to_dev(inputs.plummer_positions(n, (95, n, key)), dev) if shape == "plummer" else \
        to_dev(inputs.rng(95, n, key).random((n, 3)), dev)
    m = inputs.equal_masses(n) if mass == "equal" else inputs.lognormal_masses(n, (95, n, key, 1))
    return x, to_dev(m, dev)


def _rows64(n, dev):
    """Row indices, in chunks whose pair matrices stay small."""
    rows = torch.arange(0, n, max(1, n // ROWS), device=dev)
    return rows.split(max(1, (1 << 25) // n))


def _pairs64(x, rows, eps2):
    d = [x[rows, c, None] - x[None, :, c] for c in range(3)]
    s = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + eps2
    s[torch.arange(len(rows), device=x.device), rows] = float("inf")
    return d, s.rsqrt()


def _forces64(x, m, eps2):
    a, p = [], []
    for rows in _rows64(len(m), x.device):
        d, r = _pairs64(x, rows, eps2)
        f = r.pow(3) * m
        a.append(torch.stack([(f * d[c]).sum(1) for c in range(3)], 1))
        p.append((r * m).sum(1))
    return torch.cat(a), torch.cat(p)


def _vjp64(x, m, eps2, w, v):
    gx, gm = [], []
    for rows in _rows64(len(m), x.device):
        d, r = _pairs64(x, rows, eps2)
        r3, mk = r.pow(3), m[rows, None]
        wk = sum(w[rows, c, None] * d[c] for c in range(3))
        wj = sum(w[None, :, c] * d[c] for c in range(3))
        u = 3 * r * r * (m * wk - mk * wj)
        s = -(r3 * wj).sum(1)
        if v is not None:
            u = u + m * v[rows, None] + mk * v
            s = s + (r * v).sum(1)
        gx.append(torch.stack([(r3 * (m * w[rows, c, None] - mk * w[None, :, c] - u * d[c])).sum(1)
                               for c in range(3)], 1))
        gm.append(s)
    return torch.cat(gx), torch.cat(gm)


def _off(got, want, n):
    g = got[::max(1, n // ROWS)].double()
    return float((g - want).norm() / want.norm())


def forward_error(nb, n, mass, shape, eps2):
    dev, e = need_gpu(), []
    for key in range(2):
        x, m = _system(n, mass, shape, key, dev)
        want = _forces64(x.double(), m.double(), eps2)
        got = nb.forces(x, m, eps2)
        e.append([_off(g, w, n) for g, w in zip(got, want)])
    return [sum(c) / len(e) for c in zip(*e)]


def adjoint_error(nb, n, mass, shape, with_v, eps2):
    dev, e = need_gpu(), []
    for key in range(2):
        x, m = _system(n, mass, shape, key, dev)
        w = to_dev(inputs.normal((n, 3), (95, n, key, 2)), dev)
        v = to_dev(inputs.normal((n,), (95, n, key, 3)), dev) if with_v else None
        want = _vjp64(x.double(), m.double(), eps2, w.double(), None if v is None else v.double())
        got = nb.forces_backward(x, m, eps2, w, v)
        e.append([_off(g, t, n) for g, t in zip(got, want)])
    return [sum(c) / len(e) for c in zip(*e)]


@pytest.mark.parametrize("n,mass,shape,plain", FORWARD)
def test_forward(nb, n, mass, shape, plain):
    got = forward_error(nb, n, mass, shape, 1e-2)
    print(f"[sum error] forward {n} {mass} {shape}: {got} plain {plain}", flush=True)
    assert all(g <= 1.02 * q for g, q in zip(got, plain)), (got, plain)


@pytest.mark.parametrize("n,mass,shape,with_v,plain", ADJOINT)
def test_adjoint(nb, n, mass, shape, with_v, plain):
    got = adjoint_error(nb, n, mass, shape, with_v, 1e-2)
    print(f"[sum error] adjoint {n} {mass} {shape} {with_v}: {got} plain {plain}", flush=True)
    assert all(g <= 1.02 * q for g, q in zip(got, plain)), (got, plain)
