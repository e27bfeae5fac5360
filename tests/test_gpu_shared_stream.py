"""Leap-frog calls at the row-group sizes hold no library memory that another
call could touch: host threads that share a stream, and a captured call beside
later calls on the stream it was captured on, keep the bits of a call alone."""

import threading

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


def _state(nb, n, key, dev):
    x = to_dev(inputs.plummer_positions(n, (91, n, key)), dev)
    v = to_dev(inputs.normal((n, 3), (91, n, key, 1)), dev) * 0.1
    m = to_dev(inputs.lognormal_masses(n, (91, n, key, 2)), dev)
    return x, v, nb.forces(x, m, 1e-3, potential=False)[0], m


@pytest.mark.parametrize("n", [130, 2000, 4400, 6001])
def test_threads_on_one_stream(nb, n):
    dev = need_gpu()
    steps = 64
    states = [_state(nb, n, k, dev) for k in range(2)]
    want = []
    for x, v, a, m in states:
        want.append([t.clone() for t in (x, v, a)])
        nb.leapfrog_(*want[-1], m, 1e-3, 1e-2, steps)
    torch.cuda.synchronize()
    start, errors = threading.Barrier(2), []

    def work(k):
        try:
            x, v, a, m = states[k]
            for _ in range(8):
                got = [t.clone() for t in (x, v, a)]
                start.wait(timeout=60)
                nb.leapfrog_(*got, m, 1e-3, 1e-2, steps)
                if not all(torch.equal(t, w) for t, w in zip(got, want[k])):
                    errors.append(f"thread {k}: other bits")
        except Exception as e:  # reported below
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=120)
    assert not any(t.is_alive() for t in threads)
    assert not errors, errors[:3]


@pytest.mark.parametrize("steps", [3, 4])
def test_captured_call_holds_no_library_memory(nb, steps):
    # between the replays: a reverse sweep that needs a larger buffer on the
    # stream of the capture, its workspace given back, and a call beside the replay
    dev = need_gpu()
    n = 2000
    x, v, a, m = _state(nb, n, 5, dev)
    want = [t.clone() for t in (x, v, a)]
    nb.leapfrog_(*want, m, 1e-3, 1e-2, steps)
    got = [t.clone() for t in (x, v, a)]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        nb.leapfrog_(*[t.clone() for t in (x, v, a)], m, 1e-3, 1e-2, steps)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        nb.leapfrog_(*got, m, 1e-3, 1e-2, steps)
    big = 70001
    pos = to_dev(inputs.plummer_positions(big, (91, 7)), dev).expand(2, big, 3).contiguous()
    mb, lx = to_dev(inputs.equal_masses(big), dev), to_dev(inputs.normal((big, 3), (91, 8)), dev)
    lv, lm = lx.clone(), torch.zeros(big, device=dev)
    torch.cuda.synchronize()
    for r in range(3):
        for t, src in zip(got, (x, v, a)):
            t.copy_(src)
        with torch.cuda.stream(s):
            if r == 0:
                nb.leapfrog_adjoint_(pos, mb, 1e-3, 1e-2, lx, lv, lm)
            if r == 1:
                s.synchronize()
                nb.release_workspace()
            beside = [t.clone() for t in (x, v, a)]
        torch.cuda.synchronize()
        g.replay()
        with torch.cuda.stream(s):
            nb.leapfrog_(*beside, m, 1e-3, 1e-2, steps)
        torch.cuda.synchronize()
        assert all(torch.equal(t, w) for t, w in zip(got, want)), r
        assert all(torch.equal(t, w) for t, w in zip(beside, want)), r


def test_captured_reverse_sweep_keeps_its_buffer(nb):
    # 16 n bytes for the row-group adjoint too: at 65,536 bodies the 1 MiB that
    # the captured small sweep already holds, so the buffer stays where it is
    dev = need_gpu()
    n, big, steps = 2000, 1 << 16, 3
    pos = to_dev(inputs.normal((steps + 1, n, 3), (92, 0)), dev)
    m = to_dev(inputs.lognormal_masses(n, (92, 1)), dev)
    lx, lv = (to_dev(inputs.normal((n, 3), (92, 2 + k)), dev) for k in range(2))
    lm = torch.zeros(n, device=dev)
    want = [t.clone() for t in (lx, lv, lm)]
    nb.leapfrog_adjoint_(pos, m, 1e-3, 1e-2, *want)
    got = [t.clone() for t in (lx, lv, lm)]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        nb.leapfrog_adjoint_(pos, m, 1e-3, 1e-2, *[t.clone() for t in (lx, lv, lm)])
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        nb.leapfrog_adjoint_(pos, m, 1e-3, 1e-2, *got)
    pb = to_dev(inputs.normal((2, big, 3), (92, 5)), dev)
    mb = to_dev(inputs.equal_masses(big), dev)
    nb.set_variant(nb.BACKWARD, nb.variant_names(nb.BACKWARD).index("bwd_row_k1"))
    try:
        with torch.cuda.stream(s):
            nb.leapfrog_adjoint_(pb, mb, 1e-3, 1e-2, torch.ones_like(pb[0]), torch.ones_like(pb[0]),
                                 torch.zeros_like(mb))
        torch.cuda.synchronize()
    finally:
        nb.set_variant(nb.BACKWARD, -1)
    hold = [torch.full((1 << 18,), float("nan"), device=dev) for _ in range(8)]  # takes freed memory
    for r in range(3):
        for t, src in zip(got, (lx, lv, lm)):
            t.copy_(src)
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(t, w) for t, w in zip(got, want)), r
        assert all(bool(t.isnan().all()) for t in hold)
