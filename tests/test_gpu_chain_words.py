"""One fp32 image: the tasks of the chained kernel wait for each other's words, which are all ones until they are written."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import assert_close, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,size,classes", [(1, 33, 7), (2, 97, 1001), (3, 64, 1024), (4, 32, 1), (4, 224, 1000)])
def test_stale_words(q, size, classes):
    """Passes through a workspace of zeros, of ones and of another image's values: results of 1 x 1 to 7 x 7 last maps."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=81, batch=2, image_size=size, width_quarters=q, classes=classes)
    ref = [oracle.mobilenet_v1_forward(d["image"][i:i + 1], d["weights"]) for i in range(2)]
    model = tfx.MobileNetV1(d["weights"], batch=1, image_size=size, width_quarters=q)
    for turn, stale in enumerate((0, 255, None, None)):
        if stale is not None:
            model.workspace.fill_(stale)
        p, l = model.forward(dev(d["image"][turn % 2:turn % 2 + 1]))
        assert_close(host(l), ref[turn % 2][1], "logits, turn %d" % turn)
        assert_close(host(p), ref[turn % 2][0], "probs, turn %d" % turn)


@pytest.mark.parametrize("q,size", [(1, 64), (4, 96)])
def test_a_nan_of_all_ones_is_a_value(q, size):
    """A NaN whose bits are all ones, in the image or in a bias inside the chain, reaches every result; the next pass is right."""
    import paper_1901_05350_amd as tfx
    ones = np.array([0xffffffff], dtype=np.uint32).view(np.float32)[0]
    d = inputs.mobilenet_v1(seed=82, batch=1, image_size=size, width_quarters=q, classes=10)
    probs, logits = oracle.mobilenet_v1_forward(d["image"], d["weights"])
    model = tfx.MobileNetV1(d["weights"], batch=1, image_size=size, width_quarters=q)
    bad = d["image"].copy()
    bad[0, size // 2, size // 2, 1] = ones
    p, l = model.forward(dev(bad))
    assert np.isnan(host(l)).all() and np.isnan(host(p)).all()
    for name, block in (("pw_b", 8), ("dw_b", 12)):
        good = model.tensors[name][block].clone()
        model.tensors[name][block][3] = float(ones)
        p, l = model.forward(dev(d["image"]))
        assert np.isnan(host(l)).all() and np.isnan(host(p)).all()
        model.tensors[name][block].copy_(good)
        p, l = model.forward(dev(d["image"]))
        assert_close(host(l), logits, "logits")
        assert_close(host(p), probs, "probs")
