"""The native front of forces and forces_backward: the same results, objects
and errors as the Python path, which takes what the front declines."""

import pytest
import torch

from paper_0904_3659_amd import inputs
from tests.gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture()
def nb():
    need_gpu()
    from paper_0904_3659_amd import nbody
    nbody.lib()
    if nbody._native is None:
        pytest.skip("several devices: the Python path serves every call")
    return nbody


def _system(n, dev):
    return [to_dev(a, dev) for a in (inputs.plummer_positions(n, (85, n)), inputs.lognormal_masses(n, (85, n, 1)),
                                     inputs.normal((n, 3), (85, n, 2)), inputs.normal((n,), (85, n, 3)))]


def _python(nb, monkeypatch):
    monkeypatch.setattr(nb, "_fast_forces", None)
    monkeypatch.setattr(nb, "_fast_backward", None)


@pytest.mark.parametrize("n", [0, 1, 300, 20001])
def test_same_results(nb, n, monkeypatch):
    dev = need_gpu()
    x, m, w, v = _system(n, dev)
    a, p = torch.empty_like(x), torch.empty_like(m)
    calls = [lambda: nb.forces(x, m, 1e-4), lambda: nb.forces(x, m, 1e-4, potential=False),
             lambda: nb.forces(x, m, 1e-4, f64_sum=True), lambda: nb.forces(x, m, 1e-4, out=(a, p)),
             lambda: nb.forces(x, m, 1e-4, out=(a, None)), lambda: nb.forces_backward(x, m, 1e-4, w, v),
             lambda: nb.forces_backward(x, m, 1e-4, None, v), lambda: nb.forces_backward(x, m, 1e-4, w),
             lambda: nb.forces_backward(x, m, 1e-4, w, need_grad_m=False),
             lambda: nb.forces_backward(x, m, 1e-4, w, v, out=(a, p))]
    for k, call in enumerate(calls):
        native = [None if t is None else t.clone() for t in call()]
        with monkeypatch.context() as c:
            _python(nb, c)
            plain = call()
        for s, t in zip(native, plain):
            assert (s is None) == (t is None), k
            assert s is None or (torch.equal(s, t) and not s.requires_grad), k
    assert nb.forces(x, m, 1e-4, out=(a, p))[0] is a


def test_current_stream_is_used(nb):
    dev = need_gpu()
    x, m, w, v = _system(4000, dev)
    want = nb.forces(x, m, 1e-4)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        x2 = x.clone()
        torch.cuda._sleep(20_000_000)
        x2.mul_(1.0)
        got = nb.forces(x2, m, 1e-4)
    s.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_what_it_declines_is_refused_or_served_as_before(nb):
    dev = need_gpu()
    x, m, w, v = _system(64, dev)
    bad = [((x.cpu(), m, 1e-4), ValueError), ((x.double(), m, 1e-4), TypeError), ((x[:, :2], m, 1e-4), ValueError),
           ((x.t().contiguous().t(), m, 1e-4), ValueError), ((x, m[:-1], 1e-4), ValueError),
           ((x, m, -1.0), ValueError), ((x, m, float("nan")), ValueError), ((x, m, float("inf")), ValueError),
           ((x, None, 1e-4), TypeError)]
    for args, kind in bad:
        with pytest.raises(kind):
            nb.forces(*args)
        with pytest.raises(kind):
            nb.forces_backward(*args, w)
    with pytest.raises(ValueError):
        nb.forces(x, m, 1e-4, out=(torch.empty((63, 3), device=dev), None))
    with pytest.raises(nb.NBodyError):          # output over input: refused by the library
        nb.forces(x, m, 1e-4, out=(x, None))
    want = nb.forces(x, m, 1.0)
    for args in ((torch.nn.Parameter(x), m, 1.0), (x, m, 1), (x, m, torch.tensor(1.0))):
        got = nb.forces(*args)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    a, p = torch.empty_like(x), torch.empty_like(m)
    nb.forces(x, m, 1.0, out=[a, p])            # a list: the Python path
    assert torch.equal(a, want[0]) and torch.equal(p, want[1])
    with pytest.raises(RuntimeError):           # under vmap there is no data pointer
        torch.vmap(lambda t: nb.forces(t, m, 1.0)[0])(torch.stack([x, x]))
