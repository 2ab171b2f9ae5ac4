"""fp32 products and pointwise convolutions of K >= 256 on every kernel that takes them: what has one term, or whole numbers for
terms, comes back exact, and the epilogue keeps a bias that is not finite."""
import numpy as np
import pytest

from tests.util import dev, host

pytestmark = pytest.mark.gpu

# (M, N) that the choice gives to tiles of 128 x 128 and 64 x 64, to the kernels that split K and to the one of 16 rows; odd rows and columns
SIZES = [(1536, 1280), (3001, 1029), (700, 1500), (513, 449), (196, 128), (16, 1000)]


@pytest.mark.parametrize("m,n", SIZES)
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
def test_one_term_is_exact(m, n, ta, tb):
    """A selection of rows times a power of two, on either side: the other operand's bits, all 24 of them."""
    import paper_1901_05350_amd as tfx
    for k in (256, 515):
        rng = np.random.default_rng(m + k)
        row, power = rng.integers(0, k, m), (2.0 ** rng.integers(-3, 4, m)).astype(np.float32)
        pick = np.zeros((m, k), np.float32)
        pick[np.arange(m), row] = power
        full = rng.standard_normal((k, n)).astype(np.float32)
        a, b = np.ascontiguousarray(pick.T) if ta else pick, np.ascontiguousarray(full.T) if tb else full
        assert np.array_equal(host(tfx.tfx_matmul(dev(a), dev(b), ta, tb)), full[row] * power[:, None])
        # the selection as the right operand: (pick full)^T
        a, b = full if ta else np.ascontiguousarray(full.T), pick if tb else np.ascontiguousarray(pick.T)
        assert np.array_equal(host(tfx.tfx_matmul(dev(a), dev(b), ta, tb)), full[row].T * power)


@pytest.mark.parametrize("m,n", SIZES)
def test_whole_numbers_are_exact(m, n):
    """Products of 12-bit whole numbers whose sums of magnitudes stay below 2^24: every order of adding them is exact."""
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(m)
    a, b = np.zeros((m, 300)), rng.integers(-2100, 2101, (300, n))
    for i in range(3):  # three terms a result
        a[np.arange(m), 100 * i + rng.integers(0, 100, m)] = rng.integers(-2100, 2101, m)
    assert (np.abs(a) @ np.abs(b)).max() < 2 ** 24
    assert np.array_equal(host(tfx.tfx_matmul(dev(a), dev(b))), (a @ b).astype(np.float32))


@pytest.mark.parametrize("act", [0, 1, 2])
@pytest.mark.parametrize("n,h,co", [(64, 14, 512), (31, 13, 515), (4, 14, 512), (5, 13, 197), (1, 7, 1000)])
def test_bias_that_is_not_finite(n, h, co, act):
    """The activations keep a NaN, and take infinities to their bounds."""
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(co + act)
    x, w = rng.uniform(-1, 1, (n, h, h, 288)).astype(np.float32), (rng.standard_normal((1, 1, 288, co)) * .08).astype(np.float32)
    b = rng.standard_normal(co).astype(np.float32)
    special = {0: np.nan, 70: np.inf, 71: -np.inf, 133: np.nan, co - 1: np.nan, co - 2: -np.inf}
    for i, v in special.items():
        b[i] = v
    got = host(tfx.tfx_conv2d(dev(x), dev(w), dev(b), 1, tfx.PAD_SAME, act)).reshape(-1, co)
    rest = [i for i in range(co) if i not in special]
    for i, v in special.items():
        want = np.float32(v) if act == 0 or v != v else np.float32(np.clip(v, 0, np.inf if act == 1 else 6))
        assert np.array_equal(got[:, i], np.full(len(got), want), equal_nan=True), (i, v)
    ref = x.reshape(-1, 288).astype(np.float64) @ w[0, 0].astype(np.float64) + b
    size = np.abs(x.reshape(-1, 288)).astype(np.float64) @ np.abs(w[0, 0]).astype(np.float64) + np.abs(b)
    ref = ref if act == 0 else np.clip(ref, 0, np.inf if act == 1 else 6)
    assert np.all(np.abs(got[:, rest] - ref[:, rest]) <= 2 * 289 * 2.0 ** -24 * size[:, rest])  # 289 roundings on either side


@pytest.mark.parametrize("act", [0, 1, 2])
@pytest.mark.parametrize("n,h,co", [(64, 14, 512), (31, 13, 515), (4, 14, 512), (5, 13, 197), (1, 7, 1000)])
def test_epilogue_of_results_computed_again(n, h, co, act):
    """NaN and infinities in the image and the filter, columns that nothing but tiny weights reach, single and side by side, and a bias
    that takes a sum away again."""
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(7 * co + act)
    x, w = rng.uniform(-1, 1, (n * h * h, 288)).astype(np.float32), (rng.standard_normal((288, co)) * .08).astype(np.float32)
    b = rng.standard_normal(co).astype(np.float32)
    w[:, [2, 90] + list(range(128, 160))] *= np.float32(2.0 ** -118)
    b[[2, 90] + list(range(128, 160))] = 0
    b[40] = -np.float32(x[17].astype(np.float64) @ w[:, 40].astype(np.float64))
    x[5, 7], x[40, 100], w[9, 60] = np.nan, np.inf, -np.inf
    with np.errstate(all="ignore"):
        ref = x.astype(np.float64) @ w.astype(np.float64) + b
    size = np.nan_to_num(np.abs(x.astype(np.float64)), posinf=0) @ np.nan_to_num(np.abs(w.astype(np.float64)), posinf=0) + np.abs(b)
    ref = ref if act == 0 else np.clip(ref, 0, np.inf if act == 1 else 6)
    got = host(tfx.tfx_conv2d(dev(x.reshape(n, h, h, 288)), dev(w.reshape(1, 1, 288, co)), dev(b), 1, tfx.PAD_SAME, act)).reshape(-1, co)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf].astype(np.float32))
    fin = np.isfinite(ref)
    assert np.all(np.abs(got[fin] - ref[fin]) <= 2 * 289 * 2.0 ** -24 * size[fin] + 289 * 2.0 ** -149)  # 289 roundings on either side
    assert (got[:, 2] != 0).any() and (got[:, 128:160] != 0).any()
