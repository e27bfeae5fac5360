"""Row groups take no workspace, also where they stand in for a pair-once variant:
captured on a stream that has made no call, and refused only where that variant's
plan would be."""

import pytest
import torch

from paper_0904_3659_amd import inputs
from tests.gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    need_gpu()
    from paper_0904_3659_amd import nbody
    return nbody


@pytest.mark.parametrize("n", [1500, 4500, 6001, 10499])
def test_captured_on_a_fresh_stream(nb, n):
    dev = need_gpu()
    x, m = to_dev(inputs.plummer_positions(n, (101, n)), dev), to_dev(inputs.lognormal_masses(n, (101, n, 1)), dev)
    v = to_dev(inputs.normal((n, 3), (101, n, 2)), dev)
    a0 = nb.forces(x, m, 1e-3, potential=False)[0]
    calls = [lambda o: nb.forces(x, m, 1e-3, out=(o[0], o[3])),
             lambda o: nb.leapfrog_(o[0].copy_(x), o[1].copy_(v), o[2].copy_(a0), m, 1e-3, 1e-2, 3)]
    if n < 6200:
        calls.append(lambda o: nb.forces_backward(x, m, 1e-3, v, m, out=(o[0], o[3])))
    new = lambda: [torch.zeros((n, 3), device=dev) for _ in range(3)] + [torch.zeros(n, device=dev)]
    for k, call in enumerate(calls):
        want, got = new(), new()
        call(want)
        torch.cuda.synchronize()
        nb.release_workspace()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            call(got)
        for r in range(3):
            for t in got:
                t.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(t, w) for t, w in zip(got, want) if bool(w.any())), (k, r)
            nb.forces(x, m, 1e-3)


@pytest.mark.parametrize("n", [4500, 6001])
def test_refused_as_the_plan_would_be(nb, n, monkeypatch):
    dev = need_gpu()
    x, m = to_dev(inputs.plummer_positions(n, (102, n)), dev), to_dev(inputs.equal_masses(n), dev)
    want, grad = nb.forces(x, m, 1e-3), nb.forces_backward(x, m, 1e-3, x)
    monkeypatch.setenv("NBODY_SYM_WORKSPACE", str(16 * n * 4 - 1))
    for call in (lambda: nb.forces(x, m, 1e-3), lambda: nb.forces_backward(x, m, 1e-3, x)):
        with pytest.raises(nb.NBodyError) as e:
            call()
        assert e.value.status == 1
    monkeypatch.setenv("NBODY_SYM_WORKSPACE", str(16 * n * 4))
    assert all(torch.equal(s, t) for s, t in zip(nb.forces(x, m, 1e-3), want))
    assert all(torch.equal(s, t) for s, t in zip(nb.forces_backward(x, m, 1e-3, x), grad))
