"""fp32 networks whose second block runs in the stem's launch (block_rows.hip): maps of odd and even extents, ragged last columns, strips
of odd length, values that the split of the second pointwise product does not carry."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import assert_close, dev, host

pytestmark = pytest.mark.gpu


def features(d, batch, size, q, weights=None):
    """The map of block 2 for `batch` copies of the images in turn, and the oracle's for each image."""
    import paper_1901_05350_amd as tfx
    w = weights or d["weights"]
    ref = oracle.mobilenet_v1_forward(d["image"], w, return_activations=True)[2][4]
    model = tfx.MobileNetV1(w, batch=batch, image_size=size, width_quarters=q)
    count = d["image"].shape[0]
    image = np.concatenate([d["image"]] * ((batch + count - 1) // count))[:batch]
    return host(model.features(dev(image), 2)), ref


@pytest.mark.parametrize("q,size,batch", [(4, 224, 3), (4, 97, 15), (3, 192, 4), (3, 101, 15), (2, 66, 33), (2, 255, 3), (1, 130, 9), (1, 256, 3),
                                          (3, 256, 3), (4, 64, 36), (4, 225, 3)])
def test_two_blocks_with_the_stem(q, size, batch):
    d = inputs.mobilenet_v1(seed=93, batch=2, image_size=size, width_quarters=q, classes=10)
    got, ref = features(d, batch, size, q)
    for i in range(batch):
        assert_close(got[i], ref[i % 2], "image %d" % i)


@pytest.mark.parametrize("q", [1, 3, 4])
@pytest.mark.parametrize("what", ["a tiny value in a column", "a column of tiny values", "a large value", "all tiny", "tiny maps"])
def test_values_outside_the_split(q, what):
    size, batch = 128, 9
    d = inputs.mobilenet_v1(seed=94, batch=1, image_size=size, width_quarters=q, classes=10)
    w = {k: ([t.copy() for t in v] if isinstance(v, list) else v.copy()) for k, v in d["weights"].items()}
    f = w["pw_w"][1][0, 0]
    w["pw_b"][1][:] = 0
    if what == "a tiny value in a column":
        f[3, 5] = 3e-38
    elif what == "a column of tiny values":
        f[:, 7] = np.float32(1e-38) * np.arange(1, f.shape[0] + 1, dtype=np.float32)
    elif what == "a large value":
        f[2, 9] = 3e7
    elif what == "all tiny":
        f *= np.float32(1e-37)
    else:
        w["dw_w"][1] *= np.float32(1e-37)
        w["dw_b"][1][:] = 0
    got, ref = features(d, batch, size, q, w)
    for i in range(batch):
        # a result made of tiny values is right in its own size
        scale = np.abs(ref[0]).max(axis=(0, 1))
        scale = np.where(scale > 0, scale, 1).astype(np.float64)
        assert_close(got[i].astype(np.float64) / scale, ref[0] / scale, what)


@pytest.mark.parametrize("where", ["image", "pw_w", "dw_w", "pw_b"])
def test_nan_and_inf(where):
    """What a NaN or an infinity reaches, and nothing else."""
    size, batch, q = 128, 9, 4
    d = inputs.mobilenet_v1(seed=95, batch=2, image_size=size, width_quarters=q, classes=10)
    for value in (np.nan, np.inf, -np.inf):
        w = {k: ([t.copy() for t in v] if isinstance(v, list) else v.copy()) for k, v in d["weights"].items()}
        image = d["image"].copy()
        if where == "image":
            image[1, 40, 51, 2] = value
        else:
            w[where][1].reshape(-1, w[where][1].shape[-1] if where != "dw_w" else w[where][1].shape[2])[0, 6] = value
        got, ref = features(dict(d, image=image), batch, size, q, w)
        for i in range(batch):
            r = ref[i % 2]
            assert np.array_equal(np.isnan(got[i]), np.isnan(r)), (where, value, i)
            ok = ~np.isnan(r)
            if ok.any():  # (a NaN of the depthwise filter reaches every output)
                assert_close(got[i][ok], r[ok], "%s %s" % (where, value))


@pytest.mark.parametrize("q,size,batch,end_block", [(4, 192, 12, 13), (4, 160, 8, 9), (4, 128, 24, 11), (3, 200, 16, 10), (4, 224, 4, 9)])
def test_filters_put_in_order_by_the_same_launch(q, size, batch, end_block):
    """Tile blocks behind it, against the same blocks of one image: 4 to 7 wavefronts, filters of up to 1024 rows (read in two parts by 6)."""
    import paper_1901_05350_amd as tfx
    d = inputs.mobilenet_v1(seed=96, batch=2, image_size=size, width_quarters=q, classes=10)
    model = tfx.MobileNetV1(d["weights"], batch=batch, image_size=size, width_quarters=q)
    one = tfx.MobileNetV1(d["weights"], batch=1, image_size=size, width_quarters=q)
    model.workspace.fill_(255)
    got = host(model.features(dev(np.concatenate([d["image"]] * (batch // 2))), end_block))
    for i in (0, 1):
        ref = host(one.features(dev(d["image"][i:i + 1]), end_block))
        for j in range(i, batch, 2):
            assert_close(got[j:j + 1], ref, "image %d" % j)


@pytest.mark.parametrize("q,size,batch,end_block", [(4, 160, 48, 9), (4, 96, 64, 12), (2, 128, 64, 12)])
def test_filters_put_in_order_by_a_launch_of_their_own(q, size, batch, end_block):
    """Where the strips leave no CU idle; the tile blocks behind it against the same blocks of one image."""
    import paper_1901_05350_amd as tfx
    from test_gpu_f16_conv import launches
    d = inputs.mobilenet_v1(seed=98, batch=2, image_size=size, width_quarters=q, classes=10)
    model = tfx.MobileNetV1(d["weights"], batch=batch, image_size=size, width_quarters=q)
    one = tfx.MobileNetV1(d["weights"], batch=1, image_size=size, width_quarters=q)
    model.workspace.fill_(255)
    image = dev(np.concatenate([d["image"]] * (batch // 2)))
    got = host(model.features(image, end_block))
    assert launches(lambda: model.features(image, end_block))[1][2] == (1024, 1, 1)
    for i in (0, 1):
        ref = host(one.features(dev(d["image"][i:i + 1]), end_block))
        for j in range(i, batch, 2):
            assert_close(got[j:j + 1], ref, "image %d" % j)


def shifted(tensors, struct, names, block):
    """The named weights of one block one element behind a 16-byte boundary."""
    import torch
    for name in names:
        t = tensors[name][block]
        flat = torch.zeros(t.numel() + 1, dtype=t.dtype, device=t.device)
        flat[1:] = t.reshape(-1)
        tensors[name][block] = flat[1:].view(t.shape)
        getattr(struct, name)[block] = tensors[name][block].data_ptr()
        assert tensors[name][block].data_ptr() % 16 != 0


@pytest.mark.parametrize("half,q,size,batch", [(False, 4, 160, 6), (False, 1, 130, 9), (False, 3, 97, 15), (True, 4, 224, 10), (True, 3, 101, 47)])
@pytest.mark.parametrize("block", [0, 1])
def test_weights_off_16_bytes(half, q, size, batch, block):
    """The launch with two blocks takes them element by element: the same bits."""
    import paper_1901_05350_amd as tfx
    from util import dev16
    make, net, up = (inputs.mobilenet_v1_f16, tfx.MobileNetV1F16, dev16) if half else (inputs.mobilenet_v1, tfx.MobileNetV1, dev)
    d = make(seed=99, batch=2, image_size=size, width_quarters=q, classes=10)
    model = net(d["weights"], batch=batch, image_size=size, width_quarters=q)
    image = up(np.concatenate([d["image"]] * ((batch + 1) // 2))[:batch])
    want = host(model.features(image, 2))
    shifted(model.tensors, model.struct, ("dw_w", "dw_b", "pw_w", "pw_b"), block)
    assert np.array_equal(host(model.features(image, 2)), want)
