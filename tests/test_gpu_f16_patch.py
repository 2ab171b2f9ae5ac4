"""Depthwise-separable blocks of few pixels in one launch (block_patch_f16.hip), binary16 storage."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from test_gpu_f16_conv import dev16, end_to_end_bar, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,size,batch,blocks", [(4, 224, 1, range(1, 14)), (4, 100, 3, (1, 2, 5, 6, 7, 12, 13)), (3, 131, 2, range(1, 14)),
                                                 (2, 97, 5, range(1, 14)), (1, 37, 1, range(1, 14)), (1, 32, 9, (1, 2, 3, 13))])
def test_patch_blocks(q, size, batch, blocks):
    """Against the oracle's feature maps: every number of wavefronts and column slices, ragged patches, maps smaller than a
    patch, channel counts that fill no k-step, a NaN's positions."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1_f16(seed=80 + q, batch=batch, image_size=size, width_quarters=q, classes=10)
    d["image"][batch - 1, 17, 11, 1] = np.nan
    _, _, acts = oracle.mobilenet_v1_forward_f16(d["image"], d["weights"], return_activations=True)
    model = tfx.MobileNetV1F16(d["weights"], batch=batch, image_size=size, width_quarters=q)
    for k in blocks:
        got, ref = host(model.features(dev16(d["image"]), k)), acts[2 * k]
        assert got.shape == ref.shape and np.array_equal(np.isnan(got), np.isnan(ref)), k
        keep = ~np.isnan(ref).any(axis=-1)
        if keep.any():
            end_to_end_bar(got[keep], ref[keep], "block %d" % k, 4 if k <= 5 else 8)
