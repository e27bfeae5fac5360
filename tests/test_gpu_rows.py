"""The row-group kernels of small and middle n against the oracle: every
group size the sizes below choose, groups that straddle a tile, ragged last
tiles and groups, and the edges of the band in which they stand in for the
two-row pair-once variants."""

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
                               4499, 4500, 5003, 6209, 7001, 8200, 11999, 12000])
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
                               6199, 6200])
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
