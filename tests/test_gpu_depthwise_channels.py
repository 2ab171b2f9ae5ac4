"""3x3 depthwise convolution at channel numbers that are no multiple of a lane's (four of fp32, eight of binary16), where the last
lane of a pixel starts inside the one before it, and at addresses that no vector load is aligned to; against the oracle in float64."""
import numpy as np
import pytest
import torch

import oracle
from oracle import ACT_RELU6, PAD_SAME, PAD_VALID

pytestmark = pytest.mark.gpu


def at_odd_element(a):
    """`a` on the device, one element behind an allocation's start."""
    flat = torch.zeros(a.size + 1, dtype=torch.float16 if a.dtype == np.float16 else torch.float32, device="cuda")
    flat[1:] = torch.from_numpy(a.reshape(-1))
    return flat[1:].view(a.shape)


@pytest.mark.parametrize("c", [4, 5, 7, 8, 9, 15, 17, 30, 129])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_depthwise_any_channels(dtype, c):
    import paper_1901_05350_amd as tfx
    conv = tfx.tfx_depthwise_conv2d_f16 if dtype == np.float16 else tfx.tfx_depthwise_conv2d
    rng = np.random.default_rng(c)
    for (n, h, w), stride, pad in [((1, 3, 3), 1, PAD_VALID), ((2, 13, 6), 1, PAD_SAME), ((3, 14, 9), 2, PAD_SAME), ((64, 21, 40), 1, PAD_SAME)]:
        x = rng.uniform(-1, 1, (n, h, w, c)).astype(dtype)
        f = rng.standard_normal((3, 3, c, 1)).astype(dtype)
        b = rng.standard_normal(c).astype(dtype)
        args = [a.astype(np.float32) for a in (x, f, b)]
        want = oracle.depthwise_conv2d(*args, stride, pad, ACT_RELU6).astype(np.float64)
        size = oracle.depthwise_conv2d(*map(np.abs, args), stride, pad, 0).astype(np.float64)
        # the kernel's and the oracle's ten fp32 roundings each, and the one of the result
        limit = 20 * 2.0 ** -24 * size + (2.0 ** -11 * np.abs(want) + 2.0 ** -25 if dtype == np.float16 else 0)
        for place in (lambda a: torch.from_numpy(a).cuda(), at_odd_element):
            got = conv(place(x), place(f), place(b), stride, pad, ACT_RELU6).cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - want) <= limit), (n, h, w, stride)
