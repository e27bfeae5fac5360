"""The native front raises what the Python path raises."""

import numpy as np
import pytest
import torch

from paper_0904_3659_amd import inputs
from tests.gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(params=["native", "python"])
def nb(request, monkeypatch):
    need_gpu()
    from paper_0904_3659_amd import nbody
    nbody.lib()
    if torch.cuda.device_count() != 1:
        pytest.skip("several devices: the Python path serves every call")
    assert nbody._native is not None
    if request.param == "python":
        monkeypatch.setattr(nbody, "_fast_forces", None)
        monkeypatch.setattr(nbody, "_fast_backward", None)
    return nbody


def test_out_of_memory(nb):
    dev = need_gpu()
    n = 1 << 22  # results larger than what a cached segment of the inputs has left
    x, m = to_dev(inputs.uniform_cube(n, (96, 0)), dev), to_dev(inputs.equal_masses(n), dev)
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1e-9)  # torch's own limit: no new block
    try:
        with pytest.raises(torch.OutOfMemoryError):
            nb.forces(x, m, 1e-4)
        with pytest.raises(torch.OutOfMemoryError):
            nb.forces_backward(x, m, 1e-4, x)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)


def test_flags_without_a_truth_value(nb):
    dev = need_gpu()
    x, m = to_dev(inputs.plummer_positions(64, (96, 1)), dev), to_dev(inputs.equal_masses(64), dev)
    many = np.array([1, 2])
    with pytest.raises(ValueError):
        nb.forces(x, m, 1e-4, potential=many)
    with pytest.raises(ValueError):
        nb.forces_backward(x, m, 1e-4, x, need_grad_m=many)
    out = (torch.empty_like(x), torch.empty_like(m))  # given results: the flag is not looked at
    want = nb.forces(x, m, 1e-4)
    got = nb.forces(x, m, 1e-4, out=out, potential=many)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    nb.forces_backward(x, m, 1e-4, x, out=out, need_grad_m=many)
    assert nb.forces(x, m, 1e-4, potential=0)[1] is None
