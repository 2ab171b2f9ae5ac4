"""Depthwise-separable blocks of few pixels in one launch (block_patch.hip), fp32."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import assert_close, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,size,batch,blocks", [(4, 224, 2, range(2, 14)), (4, 100, 3, range(2, 14)), (3, 131, 2, range(2, 14)), (2, 97, 5, range(2, 14)),
                                                 (1, 37, 2, range(2, 14)), (1, 33, 9, (2, 3, 13)), (4, 64, 31, (12, 13)), (4, 224, 4, (2, 7, 12, 13))])
def test_patch_blocks(q, size, batch, blocks):
    """Against the oracle's feature maps: every number of rounds, wavefronts and column slices, ragged patches, maps smaller than a
    patch, channel counts that fill no round, a NaN's positions."""
    import paper_1901_05350_amd as tfx
    images = min(batch, 5)
    d = inputs.mobilenet_v1(seed=80 + q, batch=images, image_size=size, width_quarters=q, classes=10)
    d["image"][images - 1, 17, 11, 1] = np.nan
    _, _, acts = oracle.mobilenet_v1_forward(d["image"], d["weights"], return_activations=True)
    image = np.concatenate([d["image"]] * -(-batch // images))[:batch]
    model = tfx.MobileNetV1(d["weights"], batch=batch, image_size=size, width_quarters=q)
    for k in blocks:
        got, ref = host(model.features(dev(image), k))[:images], acts[2 * k]
        assert got.shape == ref.shape and np.array_equal(np.isnan(got), np.isnan(ref)), k
        keep = ~np.isnan(ref)
        if keep.any():
            assert_close(got[keep], ref[keep], "block %d" % k)


@pytest.mark.parametrize("q,size,batch,block,chain", [(4, 64, 2, 3, 16), (4, 64, 4, 8, 16), (4, 224, 8, 13, 64), (3, 200, 8, 13, 64), (1, 64, 4, 5, 16), (2, 64, 3, 10, 16)])
def test_sums_of_few_products(q, size, batch, block, chain):
    """One product of 4 and others of 2^-23 each, which vanish beside it: half of its last place is 2^-22.  Only those that are summed
    in one chain with it may be lost; all other sums are exact."""
    import paper_1901_05350_amd as tfx
    w = inputs.mobilenet_v1(seed=85, batch=1, image_size=size, width_quarters=q, classes=10)["weights"]
    c = w["pw_w"][block - 1].shape[2]
    w["pw_w"][block - 2][:] = 0  # the block's input: 4 in channel 0 and 1 in the others
    w["pw_b"][block - 2][:] = 1
    w["pw_b"][block - 2][0] = 4
    w["dw_w"][block - 1][:], w["dw_b"][block - 1][:], w["dw_w"][block - 1][1, 1] = 0, 0, 1
    w["pw_w"][block - 1][:], w["pw_b"][block - 1][:], w["pw_w"][block - 1][0, 0, 0] = 2.0 ** -23, 0, 1
    image = dev(np.zeros((batch, size, size, 3)))
    got = host(tfx.MobileNetV1(w, batch=batch, image_size=size, width_quarters=q).features(image, block)).astype(np.float64)
    print((got.min() - 4) * 2 ** 23, (got.max() - 4) * 2 ** 23, c)
    assert np.all(got >= 4 + (c - chain) * 2.0 ** -23) and np.all(got <= 4 + c * 2.0 ** -23)


@pytest.mark.parametrize("q,size,batch,blocks", [(3, 192, 2, (6, 7, 11)), (3, 224, 5, (13,)), (3, 60, 20, (7,)), (3, 64, 10, (13,))])
def test_patches_that_no_eight_xcds_share_evenly(q, size, batch, blocks):
    """10, 18 or 20 patches, whose grid is not padded to a multiple of the XCDs."""
    test_patch_blocks(q, size, batch, blocks)
