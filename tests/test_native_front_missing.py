"""A native front that does not load: every call works, and says so once."""

import os
import sys

import pytest
import torch

import paper_0904_3659_amd as package
from paper_0904_3659_amd import build as B
from paper_0904_3659_amd import nbody as nb


def test_library_loads_without_the_front(monkeypatch):
    if not os.path.exists(B.LIBRARY):
        pytest.skip("libnbody.so not built (run __graft_entry__.build())")
    monkeypatch.setattr(torch.cuda, "device_count", lambda: 1)
    monkeypatch.setattr(nb, "_RAW_STREAM", lambda index: 0)
    for name in ("_LIB", "_native", "_fast_forces", "_fast_backward"):
        monkeypatch.setattr(nb, name, None)
    monkeypatch.delattr(package, "_binding", raising=False)
    monkeypatch.setitem(sys.modules, "paper_0904_3659_amd._binding", None)  # import raises ImportError
    with pytest.warns(RuntimeWarning, match="native front"):
        first = nb.lib()
    assert nb.lib() is first and nb._native is None and nb._fast_forces is None
