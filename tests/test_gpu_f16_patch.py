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


@pytest.mark.parametrize("q,size,batch", [(4, 224, 1), (4, 131, 3), (3, 97, 2), (2, 256, 5), (1, 33, 2), (4, 64, 40), (1, 32, 700)])
def test_stem_and_first_block(q, size, batch):
    """block_rows_f16.hip against the oracle, image by image: strips of one row and of many, even and odd padding, ragged column
    tiles, an image that ends with the buffer; a NaN's and an infinity's positions."""
    import paper_1901_05350_amd as tfx
    images = min(batch, 5)
    d = inputs.mobilenet_v1_f16(seed=90 + q, batch=images, image_size=size, width_quarters=q, classes=10)
    d["image"][images - 1, size - 1, size - 1, 2] = np.nan
    d["image"][0, 0, 0, 0] = np.inf
    d["image"][0, 9, size - 1, 1] = -np.inf
    d["image"] = np.concatenate([d["image"]] * (batch // images))
    _, _, acts = oracle.mobilenet_v1_forward_f16(d["image"][:images], d["weights"], return_activations=True)
    model = tfx.MobileNetV1F16(d["weights"], batch=batch, image_size=size, width_quarters=q)
    got, ref = host(model.features(dev16(d["image"]), 1)), acts[2]
    assert np.array_equal(got.view(np.uint16).reshape(-1, images, *ref.shape[1:]).min(axis=0), got[:images].view(np.uint16))
    got = got[:images]
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).any()
    keep = ~np.isnan(ref).any(axis=-1)
    end_to_end_bar(got[keep], ref[keep], "stem and block 1", 4)
    assert (got[keep] != ref[keep]).mean() <= 0.005  # layers that round once: the last bit, now and then


@pytest.mark.parametrize("q,size,batch,blocks", [(3, 224, 17, (3, 4)), (3, 107, 90, (3, 4)), (2, 224, 6, (2,)), (2, 131, 17, (2,))])
def test_window_blocks_of_other_widths(q, size, batch, blocks):
    """block_stream_f16.hip at 3/4 and half width against the oracle's maps, first and last image: ragged patches and a NaN's
    positions."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1_f16(seed=85 + q, batch=2, image_size=size, width_quarters=q, classes=10)
    d["image"][1, 60, 37, 1] = np.nan
    _, _, acts = oracle.mobilenet_v1_forward_f16(d["image"], d["weights"], return_activations=True)
    image = np.concatenate([d["image"][:1]] * (batch - 1) + [d["image"][1:]])
    model = tfx.MobileNetV1F16(d["weights"], batch=batch, image_size=size, width_quarters=q)
    for k in blocks:
        got = host(model.features(dev16(image), k))[[0, -1]]
        ref = acts[2 * k]
        nan = np.isnan(ref).any(axis=-1)
        assert np.array_equal(np.isnan(got).any(axis=-1), nan) and nan.any()
        # layers that each round once: a few steps at the pixel's largest channel
        bound = 4 * np.spacing(np.abs(ref[~nan]).max(axis=-1, keepdims=True)).astype(np.float64)
        assert (np.abs(got[~nan].astype(np.float64) - ref[~nan].astype(np.float64)) <= bound).all()
