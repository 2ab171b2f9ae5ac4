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
