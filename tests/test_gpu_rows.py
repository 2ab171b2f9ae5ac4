"""Stem and first block of the fp32 network in one launch (block_rows.hip)."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import assert_close, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,size,batch", [(4, 224, 2), (4, 131, 3), (3, 97, 2), (2, 256, 5), (1, 33, 2), (4, 64, 40), (1, 32, 700)])
def test_stem_and_first_block(q, size, batch):
    """Image by image against the oracle: strips of one row and of many, even and odd padding, ragged column tiles, an image
    that ends with the buffer; a NaN's and an infinity's positions."""
    import paper_1901_05350_amd as tfx
    images = min(batch, 5)
    d = inputs.mobilenet_v1(seed=90 + q, batch=images, image_size=size, width_quarters=q, classes=10)
    d["image"][images - 1, size - 1, size - 1, 2] = np.nan
    d["image"][0, 0, 0, 0] = np.inf
    d["image"][0, 9, size - 1, 1] = -np.inf
    _, _, acts = oracle.mobilenet_v1_forward(d["image"], d["weights"], return_activations=True)
    model = tfx.MobileNetV1(d["weights"], batch=batch, image_size=size, width_quarters=q)
    got, ref = host(model.features(dev(np.concatenate([d["image"]] * (batch // images))), 1)), acts[2]
    bits = got.view(np.uint32).reshape(-1, images, *ref.shape[1:])
    assert np.array_equal(bits.min(axis=0), bits[0]) and np.array_equal(bits.max(axis=0), bits[0])
    got = got[:images]
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).any()
    keep = ~np.isnan(ref)
    assert_close(got[keep], ref[keep], "stem and block 1")


@pytest.mark.parametrize("q", [3, 4])
def test_wider_image_after_a_narrower_one(q):
    """The LDS of a launch follows the image's width, 73 KB at 224 pixels and 83 KB at 256: the call that a process makes first
    must not set the limit of the later ones."""
    import paper_1901_05350_amd as tfx
    for size in (224, 256, 193):
        d = inputs.mobilenet_v1(seed=96, batch=2, image_size=size, width_quarters=q, classes=10)
        _, _, acts = oracle.mobilenet_v1_forward(d["image"], d["weights"], return_activations=True)
        model = tfx.MobileNetV1(d["weights"], batch=2, image_size=size, width_quarters=q)
        assert_close(host(model.features(dev(d["image"]), 1)), acts[2], "%d pixels" % size)


@pytest.mark.parametrize("what,value", [("filter", np.nan), ("filter", np.inf), ("filter", 3.4e38), ("filter", 2.0 ** 20), ("filter", 1e-36),
                                        ("filter", 1e-43), ("column", 2.0 ** -118), ("maps", 2.0 ** -116), ("maps", 2.0 ** -131),
                                        ("maps", 2.0 ** -140)])
def test_values_outside_the_split(what, value):
    """A filter value, a whole column of the pointwise filter, or the depthwise outputs that feed a column, beyond what the split
    into bf16 parts carries."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=95, batch=2, image_size=96, classes=10)
    w = d["weights"]
    if what == "filter":
        w["pw_w"][0][0, 0, 17, 33] = value
    if what == "column":
        w["pw_w"][0][0, 0, :, 33] *= value
        w["pw_b"][0][33] = 0
    if what == "maps":
        w["dw_w"][0][:, :, 5], w["dw_b"][0][5] = np.abs(w["dw_w"][0][:, :, 5]) * value, 0
        w["pw_w"][0][0, 0, :, 33], w["pw_b"][0][33] = 0, 0
        w["pw_w"][0][0, 0, 5, 33] = 3
    _, _, acts = oracle.mobilenet_v1_forward(d["image"], w, return_activations=True)
    got, ref = host(tfx.MobileNetV1(w, batch=2, image_size=96).features(dev(d["image"]), 1)), acts[2]
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    keep = ~np.isnan(ref)
    assert_close(got[keep], ref[keep], what)
    if what != "filter":
        assert (ref[..., 33] != 0).any()
        # roundings of up to 32 products to 24 bits, or of a sum of nine to the smallest float (then times 3)
        assert np.all(np.abs(got[..., 33].astype(np.float64) - ref[..., 33]) <= np.maximum(1e-5 * value * 16, 32 * 2.0 ** -149))
