"""Binary16 products and convolutions of few tiles and a long contraction: two slices of the operands on their way in registers."""
import numpy as np
import pytest

import oracle
from util import assert_close_f16, dev16, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("m,n,k", [
    (512, 512, 704), (512, 512, 768), (512, 512, 832),      # whole slices: 11 (one set), 12, 13 (an odd one left over)
    (520, 500, 1217), (520, 500, 1281), (515, 509, 1345),   # a ragged last slice: 20 (even), 21 (odd), 22 slices
    (1030, 1020, 1344), (2000, 264, 1300)])                 # the wider tiles
def test_long_contractions(m, n, k, ta, tb):
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(m + n + k)
    a = rng.standard_normal((1,) + ((k, m) if ta else (m, k))).astype(np.float16)
    b = rng.standard_normal((1,) + ((n, k) if tb else (k, n))).astype(np.float16)
    assert_close_f16(host(tfx.tfx_batch_matmul_f16(dev16(a), dev16(b), ta, tb)), oracle.batch_matmul_f16(a, b, ta, tb), "%s" % ((m, n, k, ta, tb),))


@pytest.mark.parametrize("k", [768, 1300])
def test_the_last_values_of_a_contraction_count_once(k):
    import paper_1901_05350_amd as tfx
    a = np.zeros((1, 512, k), np.float16)
    b = np.zeros((1, k, 512), np.float16)
    for i, at in enumerate((0, 63, 64, 127, 128, k - 129, k - 65, k - 64, k - 2, k - 1)):
        a[0, :, at], b[0, at, :] = 1, 2.0 ** i
    got = host(tfx.tfx_batch_matmul_f16(dev16(a), dev16(b)))
    assert (got == 1023).all()


@pytest.mark.parametrize("n,h,w,cin,cout,f,stride", [
    (2, 20, 20, 128, 128, 3, 1), (2, 20, 20, 192, 128, 3, 1),          # whole 64-channel slices: 18, 27
    (1, 30, 30, 72, 96, 3, 2), (1, 30, 30, 88, 96, 3, 1),              # channels of 8: 11 (one set) and 13 slices
    (2, 21, 19, 85, 77, 3, 1), (1, 25, 30, 31, 130, 5, 1), (3, 17, 23, 90, 260, 3, 2)])  # ragged
def test_convolutions(n, h, w, cin, cout, f, stride):
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(h * cin)
    x = rng.uniform(-1, 1, (n, h, w, cin)).astype(np.float16)
    k = (rng.standard_normal((f, f, cin, cout)) * (2 / (f * f * cin)) ** 0.5).astype(np.float16)
    b = rng.standard_normal(cout).astype(np.float16)
    for pad in (tfx.PAD_SAME, tfx.PAD_VALID):
        got = host(tfx.tfx_conv2d_f16(dev16(x), dev16(k), dev16(b), stride, pad, tfx.ACT_RELU6))
        assert_close_f16(got, oracle.conv2d_f16(x, k, b, stride, pad, oracle.ACT_RELU6), "pad %d" % pad)
