"""fp32 convolutions whose input is split once under a tile (conv_window.hip), against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import assert_close, dev, host

pytestmark = pytest.mark.gpu

# (n, h, w, cin, cout, fh, fw, (stride_h, stride_w), pad): both tile heights, tiles over several images, a last tile of few
# pixels, one channel quad, channels that end inside 16, columns that end inside 64, each filter height, both strides
CASES = [(7, 42, 42, 24, 100, 3, 3, (1, 1), "same"), (61, 18, 18, 12, 93, 3, 3, (1, 1), "same"), (3, 104, 104, 16, 78, 3, 3, (1, 1), "valid"),
         (37, 11, 36, 44, 72, 3, 3, (1, 1), "valid"), (200, 7, 7, 32, 129, 3, 3, (1, 1), "same"), (1, 51, 51, 20, 499, 5, 5, (1, 1), "same"),
         (27, 81, 9, 20, 149, 5, 5, (1, 1), "valid"), (16, 56, 56, 64, 128, 3, 3, (2, 2), "same"), (15, 57, 55, 64, 128, 5, 3, (2, 1), "same"),
         (20, 40, 61, 64, 64, 3, 5, (1, 2), "same"), (60, 33, 35, 112, 60, 1, 3, (1, 1), "same"), (30, 39, 41, 32, 60, 2, 5, (1, 1), "valid"),
         (13, 47, 33, 16, 60, 7, 3, (1, 1), "valid")]


def pad_of(pad):
    return oracle.PAD_SAME if pad == "same" else oracle.PAD_VALID


@pytest.mark.parametrize("case", CASES)
def test_conv2d(case):
    import paper_1901_05350_amd as tfx
    n, h, w, ci, co, fh, fw, stride, pad = case
    d = inputs.conv_general(1100 + ci, n, h, w, ci, co, fh, fw)
    got = host(tfx.tfx_conv2d(dev(d["x"]), dev(d["filter"]), dev(d["bias"]), stride, pad_of(pad), oracle.ACT_RELU6))
    assert_close(got, oracle.conv2d(d["x"], d["filter"], d["bias"], stride, pad_of(pad), oracle.ACT_RELU6), "%r" % (case,))
    if case is CASES[0]:  # no bias, operands and result at addresses of no 16 bytes
        import torch
        off = lambda a: torch.cat([torch.zeros(1, device="cuda:0"), dev(a).reshape(-1)])[1:].view(a.shape)
        out = torch.zeros(got.size + 1, device="cuda:0")[1:].view(got.shape)
        tfx.tfx_conv2d(off(d["x"]), off(d["filter"]), None, stride, pad_of(pad), oracle.ACT_NONE, out=out)
        assert_close(host(out), oracle.conv2d(d["x"], d["filter"], None, stride, pad_of(pad), oracle.ACT_NONE), "unaligned")


@pytest.mark.parametrize("case", CASES[:2] + CASES[7:9])
def test_values_outside_the_split(case):
    """Inf and NaN in operands, tiny values beside ordinary ones, and operands so small that parts of them are below the
    smallest bf16."""
    import paper_1901_05350_amd as tfx
    n, h, w, ci, co, fh, fw, stride, pad = case
    d = inputs.conv_general(1150 + ci, n, h, w, ci, co, fh, fw)
    x, f, b = d["x"], d["filter"], d["bias"]
    x[n - 1, h - 1, w - 1, ci - 1] = np.nan
    x[0, 2, 2, 0] = np.inf
    x[n // 2, 0, 0, 1] = 1e-38
    f[0, 0, 1, 3] = 1e-36
    x[1], b[5] = 0, 0
    run = lambda x, b: host(tfx.tfx_conv2d(dev(x), dev(f), dev(b), stride, pad_of(pad), oracle.ACT_NONE))
    got, ref = run(x, b), oracle.conv2d(x, f, b, stride, pad_of(pad), oracle.ACT_NONE)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    fin = np.isfinite(ref)
    assert_close(got[fin], ref[fin], "special %r" % (case,))
    small = np.nan_to_num(x, nan=0, posinf=1) * np.float32(2.0 ** -115)
    up = oracle.conv2d(np.ldexp(small, 115), f, b, stride, pad_of(pad), oracle.ACT_NONE)
    assert_close(np.ldexp(run(small, np.ldexp(b, -115)), 115), up, "small %r" % (case,))


@pytest.mark.parametrize("n,h,w,ci,co,f", [(2, 42, 42, 16, 328, 3), (3, 76, 76, 216, 128, 3), (22, 31, 31, 40, 56, 5)])
def test_rounding_errors(n, h, w, ci, co, f):
    """Relative 2-norm error against float64.  An output is the sum of steps of f * 16 products each.  The k-th of n equal parts of a
    sum of independent terms is sqrt(k / n) of it in size, and a rounding adds some 2^-24 of that (an addition's at most, the half of
    what a matrix instruction, which cuts off, may): the additions of the steps come to steps / 2 such errors squared, those inside the
    steps to fewer than 2 f together.  (One chain of all products, with six roundings each 16, is over it.)"""
    import torch
    import paper_1901_05350_amd as tfx
    g = torch.Generator().manual_seed(ci)
    x, k = torch.randn((n, h, w, ci), generator=g), torch.randn((f, f, ci, co), generator=g)
    ref = torch.nn.functional.conv2d(x.double().permute(0, 3, 1, 2), k.double().permute(3, 2, 0, 1), padding=f // 2).permute(0, 2, 3, 1).numpy()
    got = host(tfx.tfx_conv2d(dev(x.numpy()), dev(k.numpy()), None, 1, tfx.PAD_SAME, tfx.ACT_NONE)).astype(np.float64)
    steps = (ci + 15) // 16 * f
    error = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print("steps %d: %.3g" % (steps, error))
    assert error <= 2.0 ** -24 * np.sqrt(2 * f + steps / 2)
