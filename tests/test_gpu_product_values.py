"""fp32 products of K >= 256 (gemm.hip and the kernels that it chooses from): edges of tiles and slices, and values of very different
size in one product.  The bound is K roundings to 24 bits of the sums of magnitudes on either side."""
import numpy as np
import pytest

from paper_1901_05350_amd import inputs  # noqa: F401
from tests.util import dev, host

pytestmark = pytest.mark.gpu


def product(a, b, ta=False, tb=False):
    import paper_1901_05350_amd as tfx
    return host(tfx.tfx_batch_matmul(dev(a), dev(b), ta, tb))


def check(a, b, ta=False, tb=False):
    got = product(a, b, ta, tb).astype(np.float64)
    a64, b64 = a.astype(np.float64), b.astype(np.float64)
    a64, b64 = a64.transpose(0, 2, 1) if ta else a64, b64.transpose(0, 2, 1) if tb else b64
    ref, size = a64 @ b64, np.abs(a64) @ np.abs(b64)
    k = a64.shape[2]
    assert np.all(np.abs(got - ref) <= 2 * k * 2.0 ** -24 * size + 2.0 ** -149 * k)
    return got, ref


def operands(rng, b, m, k, n, ta, tb):
    a, w = rng.standard_normal((b, k, m) if ta else (b, m, k)), rng.standard_normal((b, n, k) if tb else (b, k, n))
    return a.astype(np.float32), w.astype(np.float32)


# tiles of 128 and of 64, cut last tiles and slices, slices in the pipelined loop: none, one, many; rows of no multiple of 4
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("b,m,k,n", [(1, 1536, 256, 1280), (2, 1025, 289, 1153), (1, 2051, 1000, 1029), (1, 700, 300, 1500), (3, 513, 511, 449)])
def test_long_products(b, m, k, n, ta, tb):
    check(*operands(np.random.default_rng(k + 2 * ta + tb), b, m, k, n, ta, tb), ta, tb)


@pytest.mark.parametrize("n", [1280, 449])
def test_long_products_larger_values_behind_the_first_slice(n):
    """The first 32 of K, a slice of the tiled kernels: zeros, or values 2^8 ... 2^60 smaller than what follows."""
    rng = np.random.default_rng(7)
    for factor in (0.0, 2.0 ** -8, 2.0 ** -20, 2.0 ** -60):
        a, w = operands(rng, 1, 1300, 500, n, False, False)
        a[:, :, :32] *= factor
        check(a, w)
        w[:, :32] *= factor
        check(a * np.float32(1e-20), w * np.float32(1e18))


def test_long_products_lost_bits():
    """Rows that hold nothing but values far below the tile's largest, alone and beside a large one that meets a zero; whole columns of
    them (many results of a wavefront) and single ones (few)."""
    rng = np.random.default_rng(8)
    a, w = operands(rng, 1, 1300, 400, 1280, False, False)
    for row, scale in ((3, -35), (200, -48), (700, -70), (1299, -100)):
        a[0, row] *= 2.0 ** scale
    a[0, 40, :] *= 2.0 ** -40
    a[0, 40, 17], w[0, 17, 5:8] = 3, 0
    w[0, :, 900] *= 2.0 ** -45
    got, ref = check(a, w)
    assert np.all(got[0, [3, 200, 700]] != 0) and np.all(got[0, :, 900] != 0)
    # what only small values reach is as exact as the rest
    for part in (got[0, 200] / ref[0, 200], got[0, 40, 5:8] / ref[0, 40, 5:8]):
        assert np.median(np.abs(part - 1)) < 1e-5


def test_long_products_not_finite():
    rng = np.random.default_rng(9)
    a, w = operands(rng, 1, 1300, 300, 1280, False, True)
    a[0, 5, 7], a[0, 600, 290], w[0, 33, 100], a[0, 900, 3] = np.nan, np.inf, -np.inf, 3e38
    got = product(a, w, False, True)
    with np.errstate(all="ignore"):
        ref = (a.astype(np.float64) @ w.astype(np.float64).transpose(0, 2, 1)).astype(np.float32)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    fin = np.isfinite(ref)
    size = (np.nan_to_num(np.abs(a.astype(np.float64)), posinf=0) @ np.nan_to_num(np.abs(w.astype(np.float64)), posinf=0).transpose(0, 2, 1))
    assert np.all(np.abs(got[fin].astype(np.float64) - ref[fin]) <= 2 * 300 * 2.0 ** -24 * size[fin])
