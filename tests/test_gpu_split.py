"""GPU parity of the fp32 kernels that multiply three-way split operands on the bf16 matrix cores (split.h): values that the
split does not carry (Inf, NaN, magnitudes past the largest bf16, magnitudes near and below the smallest normal numbers), the
bits that only all three parts hold, and the edges of every kernel's tiles."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import assert_close, assert_close_f16, dev, dev16, host, time_ratio

pytestmark = pytest.mark.gpu

# (m, n, k): the 128 x 128, 64 x 64, 64 x 64 direct, 32 x 64 direct, 32 x 32 direct and 16 x 32 kernels of the dispatch
SIZES = [(4096, 1024, 96), (5000, 320, 40), (1100, 900, 700), (1000, 520, 300), (700, 300, 200), (64, 72, 96)]


@pytest.mark.parametrize("m,n,k", SIZES)
def test_values_outside_the_split(m, n, k):
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(900 + m)
    a = rng.standard_normal((m, k)).astype(np.float32)
    b = rng.standard_normal((k, n)).astype(np.float32)
    clean = host(tfx.tfx_matmul(dev(a), dev(b)))
    assert_close(clean, oracle.matmul(a, b), "clean")
    a[1, 3] = np.inf
    a[m // 2, 0] = np.nan
    a[m - 1, k - 1] = 3.4e38  # rounds to Inf as a bf16
    b[k - 1, :] = np.clip(b[k - 1, :], -0.9, 0.9)
    got, ref = host(tfx.tfx_matmul(dev(a), dev(b))), oracle.matmul(a, b)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    fin = np.isfinite(ref)
    scale = np.maximum(np.abs(a[:, :]).astype(np.float64) @ np.abs(b).astype(np.float64), 1)
    assert np.all(np.abs(got[fin] - ref[fin].astype(np.float64)) <= 1e-5 * scale[fin])


@pytest.mark.parametrize("m,n,k", SIZES)
@pytest.mark.parametrize("exponent", [-99, -101, -118, -126])
def test_small_magnitudes(m, n, k, exponent):
    """Rows of tiny values against columns of huge ones: results of ordinary size, which need every bit of the operands."""
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(950 + m)
    a = rng.standard_normal((m, k)).astype(np.float32)
    b = rng.standard_normal((k, n)).astype(np.float32)
    a[m - 2] = (1 + rng.random(k)) * 2.0 ** exponent
    b[:, n - 1] *= np.float32(2.0 ** 100)
    a[a == 0] = 1
    got, ref = host(tfx.tfx_matmul(dev(a), dev(b))).astype(np.float64), a.astype(np.float64) @ b.astype(np.float64)
    bound = 2e-6 * (np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64))
    assert np.all(np.abs(got - ref) <= np.maximum(bound, 1e-44))


# operands that are both small: ordinary results from small products, subnormal results, results that underflow; and tiny
# operands against ordinary ones, whose results are tiny and need every bit
SMALL_PAIRS = [(-60, -60), (-70, -70), (-75, -76), (-120, 0), (-140, 3), (10, -130), (-110, -2), (-112, 19), (-118, 21)]


@pytest.mark.parametrize("m,n,k", SIZES)
@pytest.mark.parametrize("ea,eb", SMALL_PAIRS)
def test_small_products(m, n, k, ea, eb):
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(960 + m)
    a = np.ldexp(rng.standard_normal((m, k)), ea).astype(np.float32)
    b = np.ldexp(rng.standard_normal((k, n)), eb).astype(np.float32)
    a[m // 2], b[:, n // 2] = 0, 0
    got = host(tfx.tfx_matmul(dev(a), dev(b))).astype(np.float64)
    exact, size = a.astype(np.float64) @ b.astype(np.float64), np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64)
    # k roundings to 24 bits, or to the smallest float
    assert np.all(np.abs(got - exact) <= k * np.maximum(2.0 ** -24 * size, 2.0 ** -149))


def test_small_products_conv2d():
    import paper_1901_05350_amd as tfx
    for i, (n, h, w, ci, co, f, s) in enumerate(CONVS):
        d = inputs.conv_general(1020 + i, n, h, w, ci, co, f, f)
        x, filt, bias = d["x"], d["filter"], d["bias"]
        x *= np.float32(2.0 ** -115)  # parts of these are below the smallest bf16
        x[0], filt[..., 0], bias[: co // 2] = 0, 0, 0
        bias[co // 2:] *= np.float32(2.0 ** -116)
        got = host(tfx.tfx_conv2d(dev(x), dev(filt), dev(bias), s, oracle.PAD_SAME, oracle.ACT_NONE))
        up = oracle.conv2d(np.ldexp(x, 115), filt, np.ldexp(bias, 115), s, oracle.PAD_SAME, oracle.ACT_NONE)
        assert_close(np.ldexp(got, 115), up, "%r" % (CONVS[i],))


@pytest.mark.parametrize("value", [1e-32, 1e-38, 1e-44])
@pytest.mark.parametrize("b,m,n,k,ta,tb", [(8, 1024, 1024, 1024, False, True), (1, 1100, 900, 700, False, False), (1, 700, 300, 600, True, True)])
def test_a_few_tiny_operands_cost_nothing(b, m, n, k, ta, tb, value):
    import torch
    import paper_1901_05350_amd as tfx
    x = torch.randn((b, k, m) if ta else (b, m, k), device="cuda:0")
    w = torch.randn((b, n, k) if tb else (b, k, n), device="cuda:0")
    tiny = torch.where(torch.rand_like(x) < 1e-3, torch.full_like(x, value), x)
    assert time_ratio(lambda v: tfx.tfx_batch_matmul(v, w, ta, tb), x, tiny) < 1.3


def test_every_bit_counts():
    """A product with the identity returns the operand bit for bit: hi, mid and lo together are the whole float."""
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(990)
    for m, k in ((4096, 128), (640, 512), (33, 40)):
        a = (rng.standard_normal((m, k)) * 2.0 ** rng.integers(-60, 60, (m, k))).astype(np.float32)
        assert np.array_equal(host(tfx.tfx_matmul(dev(a), dev(np.eye(k, dtype=np.float32)))), a)


# (n, h, w, cin, cout, f, stride): as SIZES, for the window view; channels a multiple of 32, of 4, of nothing
CONVS = [(30, 58, 57, 32, 128, 3, 1), (30, 58, 57, 36, 120, 3, 1), (20, 58, 57, 33, 130, 3, 1), (8, 56, 56, 64, 64, 3, 1),
         (3, 30, 31, 250, 130, 3, 1), (2, 27, 28, 256, 250, 3, 1), (4, 40, 40, 33, 65, 5, 1), (9, 33, 34, 16, 40, 3, 2)]


@pytest.mark.parametrize("case", CONVS)
def test_conv2d_values_outside_the_split(case):
    import paper_1901_05350_amd as tfx
    n, h, w, ci, co, f, s = case
    d = inputs.conv_general(1000 + ci, n, h, w, ci, co, f, f)
    x = d["x"]
    args = (d["filter"], d["bias"], s, oracle.PAD_SAME, oracle.ACT_NONE)
    run = lambda: host(tfx.tfx_conv2d(dev(x), dev(args[0]), dev(args[1]), s, oracle.PAD_SAME, oracle.ACT_NONE))
    assert_close(run(), oracle.conv2d(x, *args), "clean %r" % (case,))
    x[n - 1, h - 1, w - 1, ci - 1] = np.nan
    x[0, 2, 2, 0] = np.inf
    x[n // 2, 0, 0, 1] = 1e-38
    got, ref = run(), oracle.conv2d(x, *args)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    fin = np.isfinite(ref)
    assert_close(got[fin], ref[fin], "special %r" % (case,))


# binary16 through the kernels whose wavefronts split K (gemm_direct.hip): pairs of rows / columns at odd ends, both tile sizes
HALVES = [(1, 1025, 1023, 130), (1, 131, 901, 258), (2, 333, 515, 512), (1, 700, 642, 64), (1, 129, 2050, 48), (3, 65, 67, 96)]


@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
def test_matmul_f16_split_over_wavefronts(ta, tb):
    import paper_1901_05350_amd as tfx
    for i, (b, m, n, k) in enumerate(HALVES):
        d = inputs.batch_matmul_f16(seed=1100 + i, batch=b, m=m, n=n, k=k, transpose_a=ta, transpose_b=tb, bias=True)
        got = host(tfx.tfx_batch_matmul_f16(dev16(d["a"]), dev16(d["b"]), ta, tb, dev16(d["bias"]), oracle.ACT_RELU))
        assert_close_f16(got, oracle.batch_matmul_f16(d["a"], d["b"], ta, tb, d["bias"], oracle.ACT_RELU), "%r" % ((b, m, n, k),))


# tiles of a long contraction (128 x 128), of one round over the CUs (64 x 128) and of an output of few columns (64 x 64):
# (batch, m, n, k, transpose_a, transpose_b)
TILES_F16 = [(18, 325, 325, 1030, False, False), (12, 136, 592, 489, False, False), (21, 202, 220, 259, False, True),
             (24, 513, 40, 136, False, True)]


@pytest.mark.parametrize("case", TILES_F16)
def test_matmul_f16_tiles(case):
    import paper_1901_05350_amd as tfx
    b, m, n, k, ta, tb = case
    d = inputs.batch_matmul_f16(seed=1200 + n, batch=b, m=m, n=n, k=k, transpose_a=ta, transpose_b=tb, bias=True)
    got = host(tfx.tfx_batch_matmul_f16(dev16(d["a"]), dev16(d["b"]), ta, tb, dev16(d["bias"]), oracle.ACT_RELU))
    assert_close_f16(got, oracle.batch_matmul_f16(d["a"], d["b"], ta, tb, d["bias"], oracle.ACT_RELU), "%r" % (case,))


@pytest.mark.parametrize("case", [(2, 56, 56, 32, 64, 3, 1), (3, 39, 39, 176, 175, 1, 1), (4, 37, 37, 184, 87, 3, 1), (3, 20, 20, 398, 192, 5, 1),
                                  (4, 39, 41, 54, 71, 3, 2), (5, 28, 28, 16, 2, 3, 1)])
def test_conv2d_f16_split_over_wavefronts(case):
    import paper_1901_05350_amd as tfx
    n, h, w, ci, co, f, s = case
    d = inputs.conv_general(1150 + ci, n, h, w, ci, co, f, f)
    d = {key: (v * (30 if key == "bias" else 1)).astype(np.float16) for key, v in d.items()}
    got = host(tfx.tfx_conv2d_f16(dev16(d["x"]), dev16(d["filter"]), dev16(d["bias"]), s, oracle.PAD_SAME, oracle.ACT_RELU6))
    assert_close_f16(got, oracle.conv2d_f16(d["x"], d["filter"], d["bias"], s, oracle.PAD_SAME, oracle.ACT_RELU6), "%r" % (case,))


# gemm_thin.hip: one or two column blocks, several groups of them, every depth, k at and beside a k-step, rows that end a tensor
THIN = [(1, 200, 151, 3, 24, 1), (2, 160, 157, 8, 16, 1), (3, 112, 113, 15, 33, 1), (2, 71, 73, 17, 130, 1), (2, 150, 149, 33, 64, 2),
        (1, 701, 703, 31, 5, 1), (9, 230, 231, 40, 43, 1), (2, 401, 400, 24, 48, 2), (6, 128, 129, 100, 130, 1)]


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("case", THIN)
def test_thin_products(case, half):
    import paper_1901_05350_amd as tfx
    n, h, w, ci, co, s = case
    d = inputs.conv_general(1200 + ci, n, h, w, ci, co, 1, 1)
    if half:
        d = {key: v.astype(np.float16) for key, v in d.items()}
    x = d["x"]
    x[0, 0, 0, 0], x[n - 1, h - 1, w - 1, ci - 1], x[0, h // 2 // s * s, s, 0] = np.nan, np.inf, -np.inf
    up, conv, ref = (dev16, tfx.tfx_conv2d_f16, oracle.conv2d_f16) if half else (dev, tfx.tfx_conv2d, oracle.conv2d)
    got = host(conv(up(x), up(d["filter"]), up(d["bias"]), s, oracle.PAD_VALID, oracle.ACT_NONE))
    want = ref(x, d["filter"], d["bias"], s, oracle.PAD_VALID, oracle.ACT_NONE)
    assert np.array_equal(np.isfinite(got), np.isfinite(want))
    fin = np.isfinite(want)
    (assert_close_f16 if half else assert_close)(got[fin], want[fin], "%r" % (case,))


# gemm_thin.hip over a batch and with A stored [K,M]: many small matrices, so that it is the kernel taken; tiles of 32 rows and 32
# or 64 columns, k at and beside a k-step and a vector load: (batch, m, n, k)
THIN_BATCH = [(3000, 33, 65, 16), (3000, 31, 64, 17), (2500, 32, 33, 32), (9000, 64, 5, 3), (700, 65, 130, 7), (5000, 34, 31, 15),
              (6000, 33, 31, 30), (400, 129, 96, 1), (1, 2049, 2047, 9), (3, 1025, 1000, 2), (1, 16, 100003, 24)]


@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
def test_thin_products_of_a_batch(ta, tb):
    import paper_1901_05350_amd as tfx
    for i, (b, m, n, k) in enumerate(THIN_BATCH):
        rng = np.random.default_rng(1300 + i)
        x = rng.uniform(-1, 1, (b, k, m) if ta else (b, m, k)).astype(np.float32)
        w = rng.uniform(-1, 1, (b, n, k) if tb else (b, k, n)).astype(np.float32)
        x.reshape(-1)[-1], w.reshape(-1)[-1] = np.inf, -2.0  # the last element of each operand, where a load must not reach past it
        got, ref = host(tfx.tfx_batch_matmul(dev(x), dev(w), ta, tb)), oracle.batch_matmul(x, w, ta, tb)
        assert np.array_equal(np.isfinite(got), np.isfinite(ref)), (b, m, n, k)
        fin = np.isfinite(ref)
        assert_close(got[fin], ref[fin], "%r ta=%d tb=%d" % ((b, m, n, k), ta, tb))


def fp32_instructions(x, w):
    """What the fp32 matrix instructions accumulate: one product at a time, rounded to fp32."""
    acc = np.zeros((len(x), w.shape[1]), np.float32)
    for k in range(len(w)):
        acc = (acc + x[:, k:k + 1].astype(np.float64) * w[k].astype(np.float64)).astype(np.float32)
    return acc


@pytest.mark.parametrize("uniform", [False, True])
@pytest.mark.parametrize("m,n,k", [(4096, 2048, 96), (4096, 1024, 640), (5000, 320, 40), (1100, 900, 700), (1000, 520, 300), (700, 300, 200),
                                   (700, 300, 2100), (2048, 1100, 16)])
def test_error_against_float64_is_no_larger_than_with_fp32_instructions(m, n, k, uniform):
    import paper_1901_05350_amd as tfx
    rng = np.random.default_rng(1500 + k)
    draw = (lambda s: rng.random(s)) if uniform else rng.standard_normal
    x, w = draw((m, k)).astype(np.float32), draw((k, n)).astype(np.float32)
    rows = slice(m // 2, m // 2 + 96)
    got, exact = host(tfx.tfx_matmul(dev(x), dev(w)))[rows], x[rows].astype(np.float64) @ w.astype(np.float64)
    error = lambda v: np.linalg.norm(v - exact) / np.linalg.norm(exact)
    assert error(got) <= 1.05 * error(fp32_instructions(x[rows], w))  # (5 %: sampling of 96 rows)


@pytest.mark.parametrize("ta,tb", [(False, False), (True, True)])
@pytest.mark.parametrize("b,m,n", [(1, 700, 642), (16, 513, 260), (40, 17, 31), (2, 1500, 1030)])
def test_few_products_are_as_accurate_as_fp32(b, m, n, ta, tb):
    """One product is rounded once, as the hardware's fp32 multiplication rounds it; k of them at most k times."""
    import paper_1901_05350_amd as tfx
    for k in (1, 2, 3, 4):
        rng = np.random.default_rng(1400 + k)
        x, w = rng.standard_normal((b, m, k)).astype(np.float32), rng.standard_normal((b, k, n)).astype(np.float32)
        args = [dev(x.transpose(0, 2, 1)) if ta else dev(x), dev(w.transpose(0, 2, 1)) if tb else dev(w)]
        got = host(tfx.tfx_batch_matmul(*args, ta, tb))
        if k == 1:
            assert np.array_equal(got, x * w)
        exact, size = x.astype(np.float64) @ w.astype(np.float64), np.abs(x).astype(np.float64) @ np.abs(w).astype(np.float64)
        assert np.all(np.abs(got - exact) <= k * 2.0 ** -24 * size), k


def test_few_products_conv2d():
    """2 x 2 and 1 x 1 filters of few channels: outputs of one to four products."""
    import paper_1901_05350_amd as tfx
    for i, (n, hw, ci, co, f, s) in enumerate([(4, 60, 1, 40, 1, 2), (8, 90, 1, 33, 2, 1), (2, 41, 3, 70, 1, 2), (3, 30, 2, 17, 1, 2)]):
        d = inputs.conv_general(1450 + i, n, hw, hw, ci, co, f, f)
        got = host(tfx.tfx_conv2d(dev(d["x"]), dev(d["filter"]), None, s, oracle.PAD_VALID, oracle.ACT_NONE))
        rows = np.stack([d["x"][:, a:hw - f + 1 + a:s, b:hw - f + 1 + b:s] for a in range(f) for b in range(f)], 3).astype(np.float64)
        rows = rows.reshape(rows.shape[:3] + (f * f * ci,))
        flat = d["filter"].reshape(f * f * ci, co).astype(np.float64)
        assert np.all(np.abs(got - rows @ flat) <= f * f * ci * 2.0 ** -24 * (np.abs(rows) @ np.abs(flat)) + 1e-45)


@pytest.mark.parametrize("b,m,n,ta,tb", [(16, 2048, 2048, False, False), (4, 4096, 4096, True, False), (32, 1024, 1024, False, True),
                                         (1, 4096, 4096, True, True)])
def test_short_contraction_runs_at_the_speed_of_its_output(b, m, n, ta, tb):
    """The product's time is that of writing the result: at most twice that of filling it (1.0 ... 1.6 measured)."""
    import torch
    import paper_1901_05350_amd as tfx
    out = torch.empty((b, m, n), device="cuda:0")

    def us(call):
        call()
        best = 1e30
        for _ in range(5):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(10):
                call()
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end) * 100)
        return best

    fill = us(lambda: out.fill_(1.0))
    for k in (1, 4, 8, 16):
        x = torch.rand((b, k, m) if ta else (b, m, k), device="cuda:0")
        w = torch.rand((b, n, k) if tb else (b, k, n), device="cuda:0")
        got = us(lambda: tfx.tfx_batch_matmul(x, w, ta, tb, out))
        assert got <= 2 * fill, "k=%d: %.1f us, fill %.1f us" % (k, got, fill)
