"""binary16 convolutions to at most 32 channels over many pixels (tiles of 128 x 32, conv_gemm_f16.hip): every loader, last tiles ragged."""
import numpy as np
import pytest

import oracle
from util import dev16, host

pytestmark = pytest.mark.gpu

# Ci of a multiple of 64, of 8, of neither; the last column one, inside a piece of eight, and the tile's last
CASES = [(34, 64, 64, 128, 16, 3, 1), (19, 79, 81, 64, 32, 3, 1), (24, 90, 91, 16, 24, 3, 1), (21, 111, 109, 48, 32, 3, 2),
         (25, 50, 50, 162, 31, 3, 1), (8, 105, 105, 18, 12, 3, 1), (31, 62, 63, 17, 1, 5, 1), (9, 87, 87, 96, 25, 5, 1)]


@pytest.mark.parametrize("n,h,w,ci,co,f,stride", CASES)
def test_whole_numbers(n, h, w, ci, co, f, stride):
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(ci + co)
    # up to 2 and up to 1: every sum of at most 2500 products is exact in fp32; what exceeds a half's 2048 is rounded once
    x, wt = rng.integers(-2, 3, (n, h, w, ci)).astype(np.float16), rng.integers(-1, 2, (f, f, ci, co)).astype(np.float16)
    b = rng.integers(-3, 4, co).astype(np.float16)
    got = host(tfx.tfx_conv2d_f16(dev16(x), dev16(wt), dev16(b), stride, tfx.PAD_SAME, tfx.ACT_NONE))
    image = [0, n - 1]
    ref = oracle.conv2d(x[image].astype(np.float32), wt.astype(np.float32), b.astype(np.float32), stride, tfx.PAD_SAME, tfx.ACT_NONE).astype(np.float16)
    assert np.array_equal(got[image], ref)
