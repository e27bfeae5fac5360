"""The row-group kernels of small and middle n against the oracle: every
group size the sizes below choose, groups that straddle a tile, ragged last
tiles and groups, and the edges of the band in which they stand in for the
two-row pair-once variants.  Above it: one-wave pair-once blocks with a tile
per wave, ragged last blocks, odd and even block counts, the edges of their
range.  Ensembles on the same blocks."""

import numpy as np
import pytest
import torch

from oracle import reference as R
from paper_0904_3659_amd import inputs
from tests.gpu_util import assert_parity, host, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    need_gpu()
    from paper_0904_3659_amd import nbody
    return nbody


@pytest.mark.parametrize("n", [1, 2, 5, 8, 63, 64, 65, 127, 255, 257, 513, 1021, 1600, 2501, 3503, 4096,
                               4499, 4500, 5003, 6209, 7001, 8200, 10499, 10500, 11999, 12000, 12545,
                               18001, 39999, 40000, 49999])
@pytest.mark.parametrize("eps2", [0.0, 1e-4])
def test_forward(nb, n, eps2):
    dev = need_gpu()
    x = inputs.plummer_positions(n, (71, n))
    m = inputs.lognormal_masses(n, (71, n, 1))
    xd, md = to_dev(x, dev), to_dev(m, dev)
    a1 = torch.full((n + 9, 3), 7.0, device=dev)
    p1 = torch.full((n + 9,), 7.0, device=dev)
    nb.forces(xd, md, eps2, out=(a1[:n], p1[:n]))
    a2, _ = nb.forces(xd, md, eps2, potential=False)
    assert torch.equal(a1[:n], a2)                       # the same a without p
    assert bool((a1[n:] == 7.0).all()) and bool((p1[n:] == 7.0).all())
    rows = np.unique(np.concatenate([np.arange(min(n, 700)), np.arange(max(0, n - 300), n)]))
    ar, pr = R.forces_rows(x, m, eps2, rows)
    assert_parity(host(a1[:n])[rows], host(p1[:n])[rows], ar, pr, label=f"rows n={n} eps2={eps2}")


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 129, 255, 1021, 1601, 2501, 3001, 3501, 3999, 4000, 4501, 5003,
                               6199, 6200, 6401, 8193, 10499, 10500, 11777, 12000,
                               16385, 24001])
@pytest.mark.parametrize("with_v", [False, True])
def test_adjoint(nb, n, with_v):
    dev = need_gpu()
    x = inputs.plummer_positions(n, (72, n))
    m = inputs.lognormal_masses(n, (72, n, 1))
    w, v = inputs.normal((n, 3), (72, n, 2)), inputs.normal((n,), (72, n, 3))
    xd, md, wd = to_dev(x, dev), to_dev(m, dev), to_dev(w, dev)
    vd = to_dev(v, dev) if with_v else None
    gx = torch.full((n + 9, 3), 7.0, device=dev)
    gm = torch.full((n + 9,), 7.0, device=dev)
    nb.forces_backward(xd, md, 1e-4, wd, vd, out=(gx[:n], gm[:n]))
    assert bool((gx[n:] == 7.0).all()) and bool((gm[n:] == 7.0).all())
    gx2, _ = nb.forces_backward(xd, md, 1e-4, wd, vd, need_grad_m=False)
    assert torch.equal(gx[:n], gx2)
    rx, rm = R.forces_vjp(x, m, 1e-4, w, v if with_v else None)
    if n == 1:
        assert not gx[:n].any() and not gm[:n].any()
        return
    # normwise, the adjoint's tolerance of the other GPU tests
    assert np.linalg.norm(host(gx[:n]) - rx, axis=1).max() <= 1e-4 * np.linalg.norm(rx, axis=1).max()
    assert np.abs(host(gm[:n]) - rm).max() <= 1e-4 * np.abs(rm).max()


@pytest.mark.parametrize("sizes", [[1, 63, 64, 65, 128, 129, 193, 256], [257, 300, 385, 449, 511, 512, 513],
                                   [640, 705, 769, 1000, 1025, 1217, 1281, 1793, 2048]])
def test_ensemble(nb, sizes):
    # four waves share a block's tiles: last blocks of one to four row groups,
    # odd and even block counts, fewer tiles than waves
    dev = need_gpu()
    ens = inputs.ensemble(sizes + [sizes[-1]], key=(77, len(sizes)))
    a, p = nb.forces_batched(to_dev(ens.x, dev), to_dev(ens.m, dev), ens.offsets, ens.eps2)
    a2, _ = nb.forces_batched(to_dev(ens.x, dev), to_dev(ens.m, dev), ens.offsets, ens.eps2)
    assert torch.equal(a, a2)
    ar, pr = R.forces_batched(ens.offsets, ens.x, ens.m, ens.eps2)
    assert_parity(host(a), host(p), ar, pr, label=f"ensemble {sizes}")


@pytest.mark.parametrize("n", [1, 130, 2501, 5003, 11999])
@pytest.mark.parametrize("steps", [1, 2, 3, 4])
def test_leapfrog_is_the_composed_calls(nb, n, steps):
    # one launch per step, the positions alternating between the caller's
    # array and a second buffer: bitwise the separate calls, ending in x
    dev = need_gpu()
    x = to_dev(inputs.plummer_positions(n, (73, n)), dev)
    v = to_dev(inputs.plummer_velocities(host(x).astype(np.float32), (73, n, 1)), dev)
    m = to_dev(inputs.lognormal_masses(n, (73, n, 2)), dev)
    dt, eps2 = 1e-2, 1e-3
    a, _ = nb.forces(x, m, eps2)
    x1, v1, a1 = x.clone(), v.clone(), a.clone()
    hist = torch.empty((steps, n, 3), device=dev)
    nb.leapfrog_(x1, v1, a1, m, eps2, dt, steps, x_hist=hist)
    for t in range(steps):
        nb.kick_drift_(x, v, a, -0.5 * dt, dt)
        assert torch.equal(hist[t], x), t
        a, _ = nb.forces(x, m, eps2, potential=False)
        nb.axpy_(v, a, -0.5 * dt)
    assert torch.equal(x1, x) and torch.equal(v1, v) and torch.equal(a1, a)


@pytest.mark.parametrize("n", [1, 130, 2501, 4500, 6199])
@pytest.mark.parametrize("steps", [1, 2, 3])
@pytest.mark.parametrize("flags", [0, 1, 2, 3])
def test_leapfrog_adjoint_is_the_composed_calls(nb, n, steps, flags):
    dev = need_gpu()
    pos = to_dev(np.stack([inputs.plummer_positions(n, (74, n, t)) for t in range(steps + 1)]), dev)
    m = to_dev(inputs.lognormal_masses(n, (74, n, 9)), dev)
    lx, lv = (to_dev(inputs.normal((n, 3), (74, n, 10 + k)), dev) for k in (0, 1))
    lm = to_dev(inputs.normal((n,), (74, n, 12)), dev)
    dt, eps2 = 1e-2, 1e-3
    lx1, lv1, lm1 = lx.clone(), lv.clone(), lm.clone()
    nb.leapfrog_adjoint_(pos, m, eps2, dt, lx1, lv1, lm1, flags=flags)

    def kick(t, c):
        gx, gm = nb.forces_backward(pos[t], m, eps2, lv)
        nb.axpy_(lx, gx, c)
        nb.axpy_(lm, gm, c)

    if flags & nb.LEAPFROG_FINAL:
        kick(steps, -0.5 * dt)
    for t in range(steps, 0, -1):
        nb.axpy_(lv, lx, dt)
        kick(t - 1, -0.5 * dt if flags & nb.LEAPFROG_INITIAL and t == 1 else -dt)
    assert torch.equal(lx1, lx) and torch.equal(lv1, lv) and torch.equal(lm1, lm)


def test_leapfrog_captured_on_a_fresh_stream(nb):
    # no eager call on the stream, so no second position buffer there: the
    # updates run in launches of their own, with the same bits
    dev = need_gpu()
    n, steps = 1500, 3
    x = to_dev(inputs.plummer_positions(n, (75, 0)), dev)
    v = to_dev(inputs.normal((n, 3), (75, 1)), dev)
    m = to_dev(inputs.equal_masses(n), dev)
    a, _ = nb.forces(x, m, 1e-3)
    want = [t.clone() for t in (x, v, a)]
    nb.leapfrog_(*want, m, 1e-3, 1e-2, steps)
    got = [t.clone() for t in (x, v, a)]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        nb.leapfrog_(*got, m, 1e-3, 1e-2, steps)
    for _ in range(3):
        for t, src in zip(got, (x, v, a)):
            t.copy_(src)
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(t, w) for t, w in zip(got, want))
        nb.forces(x, m, 1e-3)
        torch.cuda.synchronize()
