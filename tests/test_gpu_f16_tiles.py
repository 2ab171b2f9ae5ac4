"""binary16 products through the tiled kernel (gemm_f16.hip): operands stored with their rows along the contraction are read from
LDS with the transposing load, in every tile size."""
import numpy as np
import pytest

from util import dev16, host

pytestmark = pytest.mark.gpu

# 64 x 64, 64 x 128, 128 x 128 and 256 x 256 tiles with ragged last tiles and slices; one of a batch, one of a single slice
SIZES = [(1, 701, 513, 903), (1, 1999, 1023, 1001), (1, 2050, 330, 2051), (1, 3001, 200, 3007), (3, 650, 129, 651), (1, 2049, 40, 1025)]


@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("size", SIZES)
def test_products_of_every_layout(size, ta, tb):
    import paper_1901_05350_amd as tfx
    batch, m, k, n = size
    rng = np.random.default_rng(m + k + n)
    # whole numbers up to 3: every product and every sum of up to 1023 of them (below 2^14) is exact in fp32, one rounding is left
    a, b = (rng.integers(-3, 4, (batch, r, k)).astype(np.float16) for r in (m, n))
    put = lambda v, turn: dev16(np.ascontiguousarray(v.transpose(0, 2, 1)) if turn else v)
    got = host(tfx.tfx_batch_matmul_f16(put(a, ta), put(b, not tb), ta, tb))
    ref = np.matmul(a.astype(np.float32), b.astype(np.float32).transpose(0, 2, 1)).astype(np.float16)
    assert np.array_equal(got.view(np.uint16) & 0x7fff, ref.view(np.uint16) & 0x7fff) and np.array_equal(got, ref)
