"""The pair-once kernels at sizes where no row group stands in for them: the ring
in several groups, plain and in leap-frog calls, every variant forced above the
row bands, and the default's workspace that cannot be had."""

import os
import re

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


def _kernels_per_call(nb, call):
    """Pair kernels that one call (or leap-frog step) launches."""
    nb.profile_enable(True)
    try:
        call()
        torch.cuda.synchronize()
        return nb.profile_read(launches=True)[3]
    finally:
        nb.profile_enable(False)


def _split(name, n, slots):
    """Whether n particles have more ring offsets in a variant's blocks than `slots`
    partials (its waves times rows per lane are in its name)."""
    w, k = (int(v) for v in re.match(r"..d_sym_[ws](\d+)_k(\d+)_", name).groups())
    w = 1 if "_s2_" in name else w  # two waves share a block's rows
    return -(-n // (64 * w * k)) // 2 >= slots


def _adjoint_off(gx, gm, rx, rm):
    # normwise, the adjoint's tolerance of the other GPU tests
    assert np.linalg.norm(host(gx) - rx, axis=1).max() <= 1e-4 * np.linalg.norm(rx, axis=1).max()
    assert np.abs(host(gm) - rm).max() <= 1e-4 * np.abs(rm).max()


@pytest.mark.parametrize("n", [10501, 11777])
@pytest.mark.parametrize("slots", [7, 60])
def test_every_forward_variant_in_ring_groups(nb, n, slots, monkeypatch):
    dev = need_gpu()
    x, m = inputs.plummer_positions(n, (97, n)), inputs.lognormal_masses(n, (97, n, 1))
    rows = inputs.check_rows(n, 1024, (97, n, 2))
    ar, pr = R.forces_rows(x, m, 1e-4, rows)
    xd, md = to_dev(x, dev), to_dev(m, dev)
    monkeypatch.setenv("NBODY_SYM_WORKSPACE", str(16 * n * slots))
    names = nb.variant_names(nb.FORWARD)
    try:
        for name in [v for v in names if v.startswith("fwd_sym")]:
            print(f"[ring groups] {name} n={n}", flush=True)
            nb.set_variant(nb.FORWARD, names.index(name))
            a, p = nb.forces(xd, md, 1e-4)
            kernels = _kernels_per_call(nb, lambda: nb.forces(xd, md, 1e-4))
            a2, _ = nb.forces(xd, md, 1e-4, potential=False)
            assert torch.equal(a, a2), name
            assert_parity(host(a)[rows], host(p)[rows], ar, pr, label=f"{name} n={n}")
            assert kernels > 1 or not _split(name, n, slots), name
            assert kernels > 1 or "w1_k2" not in name  # 41 offsets, and chunks
    finally:
        nb.set_variant(nb.FORWARD, -1)


@pytest.mark.parametrize("n", [6201, 11777])
def test_every_adjoint_variant_in_ring_groups(nb, n, monkeypatch):
    dev = need_gpu()
    x, m = inputs.plummer_positions(n, (97, n, 3)), inputs.lognormal_masses(n, (97, n, 4))
    w, v = inputs.normal((n, 3), (97, n, 5)), inputs.normal((n,), (97, n, 6))
    ref, ref0 = R.forces_vjp(x, m, 1e-3, w, v), R.forces_vjp(x, m, 1e-3, w, None)
    xd, md, wd, vd = (to_dev(t, dev) for t in (x, m, w, v))
    monkeypatch.setenv("NBODY_SYM_WORKSPACE", str(16 * n * 7))
    names = nb.variant_names(nb.BACKWARD)
    try:
        for name in [s for s in names if s.startswith("bwd_sym")]:
            print(f"[ring groups] {name} n={n}", flush=True)
            nb.set_variant(nb.BACKWARD, names.index(name))
            _adjoint_off(*nb.forces_backward(xd, md, 1e-3, wd, vd), *ref)
            _adjoint_off(*nb.forces_backward(xd, md, 1e-3, wd, None), *ref0)
            k = _kernels_per_call(nb, lambda: nb.forces_backward(xd, md, 1e-3, wd, vd))
            assert k > 1 or not _split(name, n, 7), (name, k)
    finally:
        nb.set_variant(nb.BACKWARD, -1)


def test_leapfrog_in_ring_groups(nb, monkeypatch):
    # the update in the fold of the last of several ring groups, forward and
    # adjoint: bitwise the composed calls, and near the FP64 integrator
    dev = need_gpu()
    n, steps, eps2, dt = 11003, 3, 1e-4, 1e-3
    monkeypatch.setenv("NBODY_SYM_WORKSPACE", str(16 * n * 7))
    x0 = inputs.plummer_positions(n, (98, 0))
    v0, m0 = inputs.plummer_velocities(x0, (98, 1)), inputs.lognormal_masses(n, (98, 2))
    x, v, m = to_dev(x0, dev), to_dev(v0, dev), to_dev(m0, dev)
    a = nb.forces(x, m, eps2, potential=False)[0]
    got, pos = [t.clone() for t in (x, v, a)], torch.empty((steps + 1, n, 3), device=dev)
    pos[0].copy_(x)
    k = _kernels_per_call(nb, lambda: nb.leapfrog_(*got, m, eps2, dt, steps, x_hist=pos[1:]))
    assert k > 1
    for t in range(steps):
        nb.kick_drift_(x, v, a, -0.5 * dt, dt)
        assert torch.equal(pos[t + 1], x)
        nb.forces(x, m, eps2, out=(a, None), potential=False)
        nb.axpy_(v, a, -0.5 * dt)
    assert all(torch.equal(p, q) for p, q in zip(got, (x, v, a)))
    rx, _ = R.leapfrog(x0, v0, m0, eps2, dt, steps)
    assert np.abs(host(x) - rx).max() <= 1e-5 * np.abs(rx).max()
    lx, lv = (to_dev(inputs.normal((n, 3), (98, 3 + c)), dev) for c in range(2))
    lm = to_dev(inputs.normal((n,), (98, 5)), dev)
    back = [t.clone() for t in (lx, lv, lm)]
    assert _kernels_per_call(nb, lambda: nb.leapfrog_adjoint_(pos, m, eps2, dt, *back, flags=2)) > 1
    for t in range(steps, 0, -1):
        nb.axpy_(lv, lx, dt)
        gx, gm = nb.forces_backward(pos[t - 1], m, eps2, lv)
        c = -0.5 * dt if t == 1 else -dt
        nb.axpy_(lx, gx, c)
        nb.axpy_(lm, gm, c)
    assert all(torch.equal(p, q) for p, q in zip(back, (lx, lv, lm)))


@pytest.mark.parametrize("n", [12001, 45001, 50021])
def test_default_pair_once_without_workspace(nb, n):
    dev = need_gpu()
    x, m = to_dev(inputs.plummer_positions(n, (99, n)), dev), to_dev(inputs.equal_masses(n), dev)
    good, _ = nb.forces(x, m, 1e-4)
    for what, status in (("launch", 4), ("alloc", 3)):
        os.environ["NBODY_FAULT"] = what
        try:
            with pytest.raises(nb.NBodyError) as ei:
                nb.forces(x, m, 1e-4)
            assert ei.value.status == status
            with pytest.raises(nb.NBodyError) as ei:
                nb.forces_backward(x, m, 1e-4, x)
            assert ei.value.status == status
        finally:
            del os.environ["NBODY_FAULT"]
    assert torch.equal(nb.forces(x, m, 1e-4)[0], good)
