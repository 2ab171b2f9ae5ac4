"""fp32 blocks with their depthwise output in LDS (block_tile.hip): every tile form, and values that the split in two halves loses."""
import numpy as np
import pytest

from paper_1901_05350_amd import inputs
from tests.util import assert_close, dev, host, time_ratio

pytestmark = pytest.mark.gpu


# 28 x 28 in tiles of 64 pixels; 14 x 14 and 7 x 7 in tiles of 32 with the contraction in 1, 2 and 4 parts; maps of odd sizes, whose last
# patches are cut; 3 column groups; the last two: blocks with too few outputs for tiles
@pytest.mark.parametrize("q,size,batch,end_block", [(4, 224, 9, 5), (4, 224, 64, 13), (4, 224, 20, 13), (4, 233, 7, 12), (4, 161, 30, 7),
                                                    (3, 201, 33, 13), (2, 131, 61, 12), (2, 224, 12, 7), (1, 224, 40, 11)])
def test_tile_blocks(q, size, batch, end_block):
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=71 + q, batch=2, image_size=size, width_quarters=q)
    image = np.concatenate([d["image"]] * (batch // 2) + [d["image"][:batch % 2]])
    got = host(tfx.MobileNetV1(d["weights"], batch=batch, image_size=size, width_quarters=q).features(dev(image), end_block))
    one = tfx.MobileNetV1(d["weights"], batch=1, image_size=size, width_quarters=q)
    for i in (0, 1):
        ref = host(one.features(dev(d["image"][i:i + 1]), end_block))
        for j in range(i, batch, 2):
            assert_close(got[j:j + 1], ref, "image %d" % j)


@pytest.mark.parametrize("batch", [8, 64])
def test_tile_blocks_columns_of_lost_bits(batch):
    """A column whose values lie 2^-32 ... 2^-70 below its largest, which multiplies zeros: what the split loses of the others is up to
    2^-20 ... 1 of them, and the results, sums of 511 products, are theirs alone."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=75, batch=8)
    w, b = d["weights"], 7
    w["dw_w"][b][:, :, 5], w["dw_b"][b][5] = 0, 0
    cols = {33: -32, 100: -40, 101: -50, 511: -70}
    for col, scale in cols.items():
        w["pw_w"][b][0, 0, :, col] *= 2.0 ** scale
        w["pw_w"][b][0, 0, 5, col] = 0.25
        w["pw_b"][b][col] = 0
    image = np.concatenate([d["image"]] * (batch // 8))
    got = host(tfx.MobileNetV1(w, batch=batch).features(dev(image), b + 1)).astype(np.float64)
    for i in (0, 3, batch - 1):
        ref = host(tfx.MobileNetV1(w, batch=1).features(dev(image[i:i + 1]), b + 1)).astype(np.float64)
        for col, scale in cols.items():
            assert (ref[..., col] != 0).any()
            # 512 roundings of 24 bits on either side, of terms of up to 6 x 0.5
            assert np.all(np.abs(got[i, ..., col] - ref[0, ..., col]) <= 2 * 512 * 2.0 ** -24 * 3 * 2.0 ** scale), col
        assert_close(got[i:i + 1], ref, "image %d" % i)


def test_static_pass_that_fits_without_tiles_only():
    """88 images of 33 x 33: tiles in a workspace of the caller's, two launches in the static one."""
    import torch
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=77, batch=4, image_size=33, classes=10)
    model = tfx.MobileNetV1(d["weights"], batch=88, image_size=33)
    assert tfx.tfx_mobilenet_v1_variant_workspace_bytes(model.variant, 88) > tfx.tfx_mobilenet_v1_static_scratch_bytes()
    image = dev(np.concatenate([d["image"]] * 22))
    probs, logits = (torch.zeros((88, 10), dtype=torch.float32, device="cuda") for _ in range(2))
    tfx.tfx_mobilenet_v1_variant_forward_static(model.variant, image, model.struct, probs, logits)
    want = model.forward(image)
    assert_close(host(logits), host(want[1]), "logits")
    assert_close(host(probs), host(want[0]), "probs")


def test_one_weight_off_16_bytes_changes_one_block():
    """Only the block that it belongs to runs as two launches: about 1.02 times the time, 1.4 with all of them."""
    import torch
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=78, batch=8)
    image = dev(np.concatenate([d["image"]] * 8))
    model, other = (tfx.MobileNetV1(d["weights"], batch=64) for _ in range(2))
    odd = torch.zeros(1025, dtype=torch.float32, device="cuda")
    odd[1:] = other.tensors["dw_b"][12]
    other.struct.dw_b[12] = odd.data_ptr() + 4
    want, got = model.forward(image), other.forward(image)
    assert_close(host(got[1]), host(want[1]), "logits")
    ratio = time_ratio(lambda m: m.forward(image), model, other)
    assert ratio < 1.15, ratio


@pytest.mark.parametrize("size,batch", [(224, 20), (231, 25)])
def test_tile_block_of_96_channels(size, batch):
    """Six k-steps; columns of small values, whose results are computed again: one of a wavefront's 64 (a sum over its lanes, of which
    half have a second channel), and all of them."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=79, batch=2, image_size=size, width_quarters=3)
    w, b = d["weights"], 3
    w["dw_w"][b][:, :, 5], w["dw_b"][b][5] = 0, 0
    cols = {3: -40, **{i: -50 for i in range(64, 128)}}
    for col, scale in cols.items():
        w["pw_w"][b][0, 0, :, col] = np.abs(w["pw_w"][b][0, 0, :, col]) * 2.0 ** scale
        w["pw_w"][b][0, 0, 5, col] = 0.25
        w["pw_b"][b][col] = 0
    image = np.concatenate([d["image"]] * (batch // 2) + [d["image"][:batch % 2]])
    got = host(tfx.MobileNetV1(w, batch=batch, image_size=size, width_quarters=3).features(dev(image), b + 1)).astype(np.float64)
    one = tfx.MobileNetV1(w, batch=1, image_size=size, width_quarters=3)
    for i in (0, 1):
        ref = host(one.features(dev(d["image"][i:i + 1]), b + 1)).astype(np.float64)
        assert all((ref[..., col] != 0).any() for col in cols)  # (positive weights)
        for j in range(i, batch, 2):
            assert_close(got[j:j + 1], ref, "image %d" % j)
            for col, scale in cols.items():
                # 96 roundings of 24 bits on either side, of terms of up to 6 x 1
                assert np.all(np.abs(got[j, ..., col] - ref[0, ..., col]) <= 2 * 96 * 2.0 ** -24 * 6 * 2.0 ** scale), col


@pytest.mark.parametrize("q,batch,block", [(4, 8, 8), (4, 64, 8), (4, 64, 13), (3, 24, 4), (2, 64, 9), (4, 16, 4)])
def test_one_term_keeps_22_bits(q, batch, block):
    """A block that moves channels about, times powers of two: what is left of a value of 24 bits in two halves, the first of 11 bits and
    the second of 11 of the 12 that a remainder can have: half a unit of the second, 2^-23, and the rounding of the result."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=76, batch=2, width_quarters=q)
    w, b = d["weights"], block - 1
    n, stride = w["pw_w"][b].shape[3], 2 if block in (2, 4, 6, 12) else 1
    c = w["pw_w"][b].shape[2]
    rng = np.random.default_rng(block)
    row, power = rng.integers(0, c, n), 2.0 ** rng.integers(-9, 1, n)
    w["dw_w"][b][:], w["dw_b"][b][:], w["pw_w"][b][:], w["pw_b"][b][:] = 0, 0, 0, 0
    w["dw_w"][b][1 if stride == 1 else 0, 1 if stride == 1 else 0] = 1  # the value itself; at stride 2 SAME pads behind the map only
    w["pw_w"][b][0, 0, row, np.arange(n)] = power
    image = np.concatenate([d["image"]] * (batch // 2))
    model = tfx.MobileNetV1(w, batch=batch, width_quarters=q)
    x = host(model.features(dev(image), block - 1)).astype(np.float64)[:, ::stride, ::stride]
    got = host(model.features(dev(image), block)).astype(np.float64)
    want = x[..., row] * power
    assert (want > 0).any() and np.all(np.abs(got - want) <= 1.5 * 2.0 ** -23 * want)


def test_tiles_in_place_of_windows():
    """128 -> 128 with less than half a round of the window kernel's units."""
    test_tile_blocks(1, 224, 64, 9)
