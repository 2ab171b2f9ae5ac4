"""binary16 convolutions whose filter is read from LDS with the transposing load (conv_gemm_f16.hip): every tile size and loader."""
import numpy as np
import pytest

import oracle
from util import dev16, host

pytestmark = pytest.mark.gpu

# 64 x 64, 64 x 128 and 128 x 128 tiles, last ones ragged; Ci of a multiple of 64, of 8, of neither; Co ending inside 8 columns
CASES = [(3, 31, 29, 64, 72, 3), (9, 26, 25, 64, 200, 3), (9, 40, 41, 128, 136, 3), (3, 31, 29, 72, 64, 3), (6, 26, 25, 40, 200, 5),
         (9, 40, 41, 72, 136, 3), (3, 31, 29, 71, 70, 3), (9, 26, 25, 37, 199, 3), (9, 40, 41, 67, 131, 3), (5, 27, 30, 100, 41, 5)]


@pytest.mark.parametrize("n,h,w,ci,co,f", CASES)
def test_whole_numbers(n, h, w, ci, co, f):
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(ci + co)
    # up to 2 and up to 1: every sum of at most 2500 products is exact in fp32; what exceeds a half's 2048 is rounded once
    x, wt = rng.integers(-2, 3, (n, h, w, ci)).astype(np.float16), rng.integers(-1, 2, (f, f, ci, co)).astype(np.float16)
    b = rng.integers(-3, 4, co).astype(np.float16)
    got = host(tfx.tfx_conv2d_f16(dev16(x), dev16(wt), dev16(b), 1, tfx.PAD_SAME, tfx.ACT_NONE))
    image = (0, n - 1)
    ref = oracle.conv2d(x[list(image)].astype(np.float32), wt.astype(np.float32), b.astype(np.float32), 1, tfx.PAD_SAME, tfx.ACT_NONE).astype(np.float16)
    assert np.array_equal(got[list(image)], ref)
