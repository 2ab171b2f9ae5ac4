"""One image on binary16 storage: the chained kernel, whose tasks wait for each other's words."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import dev16, host

pytestmark = pytest.mark.gpu


def bar(got, ref, steps, what):
    """`steps` binary16 steps at the magnitude of the largest entry: 28 layers that each round once (8 logits, 16 probabilities)."""
    step = float(np.spacing(np.abs(ref).max().astype(np.float16)))
    err = np.abs(got.astype(np.float64) - ref.astype(np.float64)).max()
    assert err <= steps * step, (what, err / step)


@pytest.mark.parametrize("q,size,classes", [(1, 33, 7), (1, 128, 1000), (2, 97, 1001), (3, 64, 1024), (3, 192, 1000), (4, 32, 1), (4, 161, 10),
                                            (4, 224, 1000), (4, 256, 129)])
def test_one_image(q, size, classes):
    """Passes through a workspace of zeros, of ones and of another image's values; 1 x 1 to 8 x 8 last maps, every split of K."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1_f16(seed=83, batch=2, image_size=size, width_quarters=q, classes=classes)
    ref = [oracle.mobilenet_v1_forward_f16(d["image"][i:i + 1], d["weights"]) for i in range(2)]
    model = tfx.MobileNetV1F16(d["weights"], batch=1, image_size=size, width_quarters=q)
    for turn, stale in enumerate((0, 255, None, None)):
        if stale is not None:
            model.workspace.fill_(stale)
        p, l = model.forward(dev16(d["image"][turn % 2:turn % 2 + 1]))
        bar(host(l), ref[turn % 2][1], 8, "logits, turn %d" % turn)
        bar(host(p), ref[turn % 2][0], 16, "probs, turn %d" % turn)


@pytest.mark.parametrize("q,size", [(1, 64), (4, 96)])
def test_a_nan_of_all_ones_is_a_value(q, size):
    """A NaN whose bits are all ones, in the image or in a bias inside the chain, reaches every result; the next pass is right."""
    import paper_1901_05350_amd as tfx
    ones = np.array([0xffff], dtype=np.uint16).view(np.float16)[0]
    d = inputs.mobilenet_v1_f16(seed=84, batch=1, image_size=size, width_quarters=q, classes=10)
    model = tfx.MobileNetV1F16(d["weights"], batch=1, image_size=size, width_quarters=q)
    image = dev16(d["image"])
    p0, l0 = [host(t).copy() for t in model.forward(image)]
    bad = d["image"].copy()
    bad[0, size // 2, size // 2, 1] = ones
    p, l = model.forward(dev16(bad))
    assert np.isnan(host(l)).all() and np.isnan(host(p)).all()
    for name, block in (("pw_b", 8), ("dw_b", 12)):
        good = model.tensors[name][block].clone()
        model.tensors[name][block][2:4] = float("nan")
        model.tensors[name][block].view(dtype=__import__("torch").int16)[2:4] = -1
        p, l = model.forward(image)
        assert np.isnan(host(l)).all() and np.isnan(host(p)).all()
        model.tensors[name][block].copy_(good)
        p, l = model.forward(image)
        assert np.array_equal(host(l), l0) and np.array_equal(host(p), p0)


def test_waits_that_give_up(monkeypatch):
    """leave NaN, not numbers."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1_f16(seed=85, batch=1, classes=10)
    probs, logits = oracle.mobilenet_v1_forward_f16(d["image"], d["weights"])
    model = tfx.MobileNetV1F16(d["weights"], batch=1)
    image = dev16(d["image"])
    monkeypatch.setenv("TFX_CHAIN_SPIN_LIMIT", "1")
    p, l = model.forward(image)
    assert np.isnan(host(p)).all() and np.isnan(host(l)).all()
    monkeypatch.delenv("TFX_CHAIN_SPIN_LIMIT")
    p, l = model.forward(image)
    bar(host(l), logits, 8, "logits")


def test_captured_and_on_two_streams():
    import torch
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1_f16(seed=86, batch=2, image_size=160, width_quarters=4, classes=100)
    models = [tfx.MobileNetV1F16(d["weights"], batch=1, image_size=160) for _ in range(2)]
    images = [dev16(d["image"][i:i + 1]) for i in range(2)]
    want = [host(m.forward(x)[1]).copy() for m, x in zip(models, images)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        p, l = models[0].forward(images[0])
    for turn in range(4):
        l.zero_()
        graph.replay()
        assert np.array_equal(host(l), want[0]), turn
        assert np.array_equal(host(models[1].forward(images[1])[1]), want[1])
    streams = [torch.cuda.Stream() for _ in range(2)]
    for turn in range(20):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                models[i].forward(images[i])
    for i in range(2):
        assert np.array_equal(host(models[i].logits), want[i])


def test_one_image_in_a_workspace_of_two():
    import ctypes
    import torch
    import paper_1901_05350_amd as tfx
    from paper_1901_05350_amd import binding
    d = inputs.mobilenet_v1_f16(seed=87, batch=1, image_size=96, width_quarters=2, classes=10)
    probs, logits = oracle.mobilenet_v1_forward_f16(d["image"], d["weights"])
    model = tfx.MobileNetV1F16(d["weights"], batch=1, image_size=96, width_quarters=2)
    size = tfx.lib().tfx_mobilenet_v1_workspace_bytes_f16(ctypes.byref(binding.TfxVariant(96, 2, 10)), 2)
    model.workspace = torch.full((size,), 255, dtype=torch.uint8, device="cuda:0")
    p, l = model.forward(dev16(d["image"]))
    bar(host(l), logits, 8, "logits")
    bar(host(p), probs, 16, "probs")
