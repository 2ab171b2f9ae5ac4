"""One full-width fp32 image whose stem filter lies off 16-byte alignment: a first kernel that clears no task flags, so nothing
after it may wait for them."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import assert_close, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stale", [0, 1, 255])
def test_unaligned_stem_filter(stale):
    """Feature maps of blocks 4 and 5 and the whole pass for two images in turn through one workspace that starts full of
    `stale` bytes: flags that read as unset, and as set before any block has run."""
    import torch
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=71, batch=2, image_size=96, classes=10)
    w = dict(d["weights"])
    ref = [oracle.mobilenet_v1_forward(d["image"][i:i + 1], w, return_activations=True) for i in range(2)]
    flat = torch.zeros(w["conv0_w"].size + 1, device="cuda:0")
    flat[1:] = dev(w["conv0_w"]).flatten()
    w["conv0_w"] = flat[1:].view(3, 3, 3, 32)
    model = tfx.MobileNetV1(w, batch=1, image_size=96)
    assert model.struct.conv0_w % 16 == 4
    model.workspace.fill_(stale)
    for turn in range(4):
        image, (probs, logits, acts) = dev(d["image"][turn % 2:turn % 2 + 1]), ref[turn % 2]
        for block in (4, 5):
            assert_close(host(model.features(image, block)), acts[2 * block], "block %d, turn %d" % (block, turn))
        p, l = model.forward(image)
        assert_close(host(l), logits, "logits, turn %d" % turn)
        assert_close(host(p), probs, "probs, turn %d" % turn)
    assert not np.array_equal(ref[0][2][8], ref[1][2][8])
