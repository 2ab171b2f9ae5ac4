"""gemm_deep.hip: both sides of each line between its numbers of wavefronts and loads, and of its one and two column blocks."""
import numpy as np
import pytest

from util import dev, dev16, host

pytestmark = pytest.mark.gpu

# workgroups of one column block: 9, 246, 258, 321; the last has one block only
SHAPES = [(40, 33), (1300, 48), (1370, 48), (1700, 48), (5200, 16)]


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("steps", [4, 8, 16])
@pytest.mark.parametrize("m,n", SHAPES)
def test_steps(m, n, steps, half):
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(m + n + steps)
    for k in (steps * (32 if half else 16), steps * (32 if half else 16) + 1):
        # whole numbers up to 3: every sum of up to 513 products is exact in fp32 (and below 2^13, so one rounding to a half is left)
        a, b = (rng.integers(-3, 4, s).astype(np.float16 if half else np.float32) for s in ((1, m, k), (1, k, n)))
        got = host(tfx.tfx_batch_matmul_f16(dev16(a), dev16(b)) if half else tfx.tfx_batch_matmul(dev(a), dev(b)))
        assert np.array_equal(got, np.matmul(a.astype(np.float32), b.astype(np.float32)).astype(a.dtype))
