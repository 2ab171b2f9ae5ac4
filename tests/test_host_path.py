"""The binding without its native host path (csrc/call.cpp): the library is called through ctypes, with the same checks."""
import sys

import pytest

from paper_1901_05350_amd import binding


def test_entry_points_work_where_the_extension_cannot_be_loaded(monkeypatch):
    import torch
    import paper_1901_05350_amd as tfx
    monkeypatch.setattr(binding, "_call", None)
    monkeypatch.setitem(sys.modules, "paper_1901_05350_amd._call", None)  # its import raises ImportError
    monkeypatch.delattr(tfx, "_call", raising=False)
    a = torch.zeros(3, 4)
    with pytest.warns(RuntimeWarning, match="_call cannot be loaded"), pytest.raises(TypeError, match="GPU memory"):
        tfx.tfx_matmul(a, a, False, True)
    with pytest.raises(TypeError, match="rank"):  # no second warning, and the checks say what is wrong
        tfx.tfx_conv2d(a, a)


@pytest.mark.gpu
def test_results_without_the_extension(monkeypatch):
    import torch
    import paper_1901_05350_amd as tfx
    a, b = torch.randn(40, 70, device="cuda:0"), torch.randn(70, 50, device="cuda:0")
    want = tfx.tfx_matmul(a, b)
    monkeypatch.setattr(binding, "_call", None)
    monkeypatch.setitem(sys.modules, "paper_1901_05350_amd._call", None)
    monkeypatch.delattr(tfx, "_call", raising=False)
    with pytest.warns(RuntimeWarning):
        got = tfx.tfx_matmul(a, b)
    assert torch.equal(got, want)
