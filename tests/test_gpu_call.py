"""GPU test of the native host path (csrc/call.cpp): the entry points give the same bits through it and through the
Python path behind it, hand back the caller's `out`, and leave what is wrong with an argument to the Python checks."""
import numpy as np
import pytest

from util import host

pytestmark = pytest.mark.gpu


def both(monkeypatch, fn):
    """fn() through the native path and with that path declining everything."""
    from paper_1901_05350_amd import binding

    class Declines:
        def __getattr__(self, name):
            return lambda *args: None

    fast = fn()
    with monkeypatch.context() as m:
        m.setattr(binding, "_call", Declines())
        slow = fn()
    return fast, slow


@pytest.mark.parametrize("half", [False, True])
def test_native_and_python_host_paths_agree(monkeypatch, half):
    import torch
    import paper_1901_05350_amd as tfx
    dt = torch.float16 if half else torch.float32
    g = torch.Generator(device="cuda:0").manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda:0").to(dt)
    a, b, bias = rnd(3, 20, 17), rnd(3, 9, 20), rnd(9)
    x, f, fd, fb, db = rnd(2, 9, 8, 5), rnd(3, 2, 5, 6), rnd(3, 3, 5, 2), rnd(6), rnd(10)
    conv, dw, add = ((tfx.tfx_conv2d_f16, tfx.tfx_depthwise_conv2d_f16, tfx.tfx_add_f16) if half else
                     (tfx.tfx_conv2d, tfx.tfx_depthwise_conv2d, tfx.tfx_add))
    calls = [lambda: conv(x, f, fb, (2, 1), tfx.PAD_VALID, tfx.ACT_RELU), lambda: conv(x, f, stride=2),
             lambda: dw(x, fd, db, [1, 2], act=tfx.ACT_RELU6), lambda: dw(x, fd), lambda: add(x, x),
             lambda: add(x, x, out=torch.empty_like(x))]
    if half:
        calls += [lambda: tfx.tfx_batch_matmul_f16(a, b, True, True, bias, tfx.ACT_RELU),
                  lambda: tfx.tfx_batch_matmul_f16(a, b, transpose_a=True, transpose_b=1)]
    else:
        calls += [lambda: tfx.tfx_batch_matmul(a, b, True, True), lambda: tfx.tfx_matmul(a[0], b[0], 1, True)]
    for i, call in enumerate(calls):
        fast, slow = both(monkeypatch, call)
        assert fast.shape == slow.shape and fast.dtype == dt and np.array_equal(host(fast), host(slow)), i
    out = torch.empty((2, 9, 8, 6), dtype=dt, device="cuda:0")
    assert conv(x, f, out=out) is out
    with pytest.raises(TypeError, match="contiguous"):
        conv(x.transpose(1, 2), f)
    with pytest.raises(TypeError, match="out must have shape"):
        conv(x, f, out=out[:1])
    with pytest.raises(TypeError, match="contiguous"):
        conv(x.double(), f)
    with pytest.raises(tfx.TfxError):
        conv(x, rnd(3, 3, 4, 6))
    with pytest.raises(tfx.TfxError):
        conv(x, f, act=7)
