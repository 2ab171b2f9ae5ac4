"""fp32 blocks whose split filter stays in LDS (block_stream.hip): values that the split into bf16 parts does not carry."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import assert_close, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [2, 3])
@pytest.mark.parametrize("what,value", [("none", 0), ("filter", np.nan), ("filter", np.inf), ("filter", 3.4e38), ("filter", 2.0 ** 20),
                                        ("filter", 1e-36), ("filter", 1e-43), ("column", 2.0 ** -118), ("maps", 2.0 ** -116),
                                        ("maps", 2.0 ** -131), ("maps", 2.0 ** -140)])
def test_values_outside_the_split(block, what, value):
    """A filter value, a whole column of the pointwise filter, or the depthwise outputs that feed a column; 25 x 25 maps, so the
    last patches are ragged; NaNs from the image."""
    import paper_1901_05350_amd as tfx
    batch = 30  # more patches than workgroups of block_patch.hip are resident, fewer than two chains of kernels are for
    d = inputs.mobilenet_v1(seed=97, batch=2, image_size=100, classes=10)
    w, b = d["weights"], block - 1
    d["image"][1, 50, 31, 1] = np.nan
    if what == "filter":
        w["pw_w"][b][0, 0, 17, 33] = value
    if what == "column":
        w["pw_w"][b][0, 0, :, 33] *= value
        w["pw_b"][b][33] = 0
    if what == "maps":
        w["dw_w"][b][:, :, 5], w["dw_b"][b][5] = np.abs(w["dw_w"][b][:, :, 5]) * value, 0
        w["pw_w"][b][0, 0, :, 33], w["pw_b"][b][33] = 0, 0
        w["pw_w"][b][0, 0, 5, 33] = 3
    _, _, acts = oracle.mobilenet_v1_forward(d["image"], w, return_activations=True)
    image = np.concatenate([d["image"]] * (batch // 2))
    got = host(tfx.MobileNetV1(w, batch=batch, image_size=100).features(dev(image), block))
    bits = got.view(np.uint32).reshape(-1, 2, *got.shape[1:])
    assert np.array_equal(bits.min(axis=0), bits[0]) and np.array_equal(bits.max(axis=0), bits[0])
    got, ref = got[:2], acts[2 * block]
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).any()
    keep = ~np.isnan(ref)
    assert_close(got[keep], ref[keep], what)
    if what in ("column", "maps"):
        g, r = got[..., 33][keep[..., 33]], ref[..., 33][keep[..., 33]]
        assert (r != 0).any()
        # roundings of up to 128 products to 24 bits, or of a sum of nine to the smallest float (then times 3)
        assert np.all(np.abs(g.astype(np.float64) - r) <= np.maximum(1e-5 * value * 16, 128 * 2.0 ** -149))


@pytest.mark.parametrize("q,size,blocks", [(2, 224, (2, 3)), (2, 203, (2, 3)), (3, 224, (3,)), (3, 195, (3,))])
def test_other_widths(q, size, blocks):
    """3/4 and half width against the oracle's maps, first and last image: ragged patches, a NaN's positions."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=99, batch=2, image_size=size, width_quarters=q, classes=10)
    d["image"][1, 60, 37, 1] = np.nan
    _, _, acts = oracle.mobilenet_v1_forward(d["image"], d["weights"], return_activations=True)
    model = tfx.MobileNetV1(d["weights"], batch=31, image_size=size, width_quarters=q)
    image = dev(np.concatenate([d["image"][:1]] * 30 + [d["image"][1:]]))
    for k in blocks:
        got, ref = host(model.features(image, k))[[0, -1]], acts[2 * k]
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).any()
        keep = ~np.isnan(ref)
        assert_close(got[keep], ref[keep], "block %d" % k)


@pytest.mark.parametrize("q,block", [(2, 3), (3, 3), (4, 3), (4, 2)])
def test_order_of_the_passes(q, block):
    """A product of 4 in the first 32 channels, and in the next 32 pairs (1 + d) W (1 + d) - (1 - d) W (1 - d) whose large parts cancel:
    of the six bf16 products only the two of a middle with a high part are left, each 15/16 of 4's last place in sum.  The matrix
    instructions cut off what lies behind the last place: added to 4 one after the other both vanish, but one place is left of their
    sum, for an error below one."""
    import paper_1901_05350_amd as tfx
    w = inputs.mobilenet_v1(seed=98, batch=1, image_size=224, width_quarters=q, classes=10)["weights"]
    d, W = 2.0 ** -10, 15 * 2.0 ** -20
    sign = np.tile(np.float64([1, -1]), 16)
    w["pw_w"][block - 2][:], w["pw_b"][block - 2][:], w["pw_b"][block - 2][0], w["pw_b"][block - 2][32:64] = 0, 0, 4, 1 + sign * d
    w["dw_w"][block - 1][:], w["dw_b"][block - 1][:], w["dw_w"][block - 1][1, 1] = 0, 0, 1
    w["pw_w"][block - 1][:], w["pw_b"][block - 1][:] = 0, 0
    w["pw_w"][block - 1][0, 0, 0], w["pw_w"][block - 1][0, 0, 32:64] = 1, (sign * W * (1 + sign * d))[:, None]
    got = host(tfx.MobileNetV1(w, batch=31, image_size=224, width_quarters=q).features(dev(np.zeros((31, 224, 224, 3))), block))
    assert np.all(np.abs(got.astype(np.float64) - (4 + 32 * W * 2 * d)) < 2.0 ** -21)
