"""GPU parity of the kernels that take any size and alignment (gemm_deep.hip, the ragged forms of gemm.hip, gemm_f16.hip and
conv_gemm_f16.hip) at the places where they can go wrong: one element more or less than a vector load, a k-step, a slice or
a tile, the last rows of a tensor, the smallest operands, and either side of the rules that pick a kernel."""
import numpy as np
import pytest

import oracle
from paper_1901_05350_amd import inputs
from util import assert_close, assert_close_f16, dev, dev16, host

pytestmark = pytest.mark.gpu

# (batch, m, n, k)
SIZES = [(1, 1, 1, 1), (1, 1, 5, 1), (2, 3, 7, 2), (1, 7, 3, 9), (3, 15, 17, 31), (1, 17, 33, 33), (1, 16, 32, 7),
         (1, 33, 34, 257), (2, 50, 63, 129), (1, 20, 300, 1031), (1, 9, 21, 3001), (1, 640, 515, 65), (1, 700, 642, 63),
         (1, 513, 1027, 191), (3, 1031, 1025, 70), (1, 2050, 2047, 130), (1, 3100, 3001, 67), (1, 5000, 6, 70)]


@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("half", [False, True])
def test_matmul_ragged_sizes(half, ta, tb):
    import paper_1901_05350_amd as tfx
    for i, (b, m, n, k) in enumerate(SIZES):
        if m * n * k > 1 << 28 and ta != tb:      # the large ones in two of the layouts
            continue
        d = inputs.batch_matmul_f16(seed=600 + i, batch=b, m=m, n=n, k=k, transpose_a=ta, transpose_b=tb, bias=True)
        where = "matmul %r ta=%d tb=%d" % ((b, m, n, k), ta, tb)
        if half:
            got = host(tfx.tfx_batch_matmul_f16(dev16(d["a"]), dev16(d["b"]), ta, tb, dev16(d["bias"]), oracle.ACT_RELU))
            assert_close_f16(got, oracle.batch_matmul_f16(d["a"], d["b"], ta, tb, d["bias"], oracle.ACT_RELU), where)
        else:
            a, w = d["a"].astype(np.float32) / 8, d["b"].astype(np.float32) / 8
            assert_close(host(tfx.tfx_batch_matmul(dev(a), dev(w), ta, tb)), oracle.batch_matmul(a, w, ta, tb), where)


# (n, h, w, cin, cout, fh, fw, stride)
CONVS = [(1, 3, 3, 1, 1, 1, 1, 2), (1, 4, 5, 1, 9, 3, 3, 1), (1, 5, 4, 2, 3, 2, 3, 1), (2, 7, 7, 7, 8, 3, 3, 1), (1, 6, 7, 9, 15, 3, 3, 2),
         (1, 9, 9, 40, 8, 5, 5, 1), (2, 13, 11, 33, 17, 3, 3, 1), (3, 12, 12, 64, 72, 3, 3, 2), (1, 17, 15, 130, 66, 1, 1, 2),
         (8, 40, 41, 3, 20, 5, 5, 1), (5, 41, 40, 31, 65, 3, 3, 1), (6, 43, 44, 36, 130, 3, 3, 1), (4, 60, 61, 24, 56, 3, 3, 1),
         (5, 57, 55, 128, 136, 3, 3, 2), (14, 57, 57, 12, 129, 2, 2, 1), (9, 64, 63, 8, 200, 3, 1, 1), (3, 80, 81, 5, 7, 7, 7, 1)]


@pytest.mark.parametrize("pad", [oracle.PAD_SAME, oracle.PAD_VALID])
@pytest.mark.parametrize("half", [False, True])
def test_conv2d_ragged_geometries(half, pad):
    import paper_1901_05350_amd as tfx
    for i, (n, h, w, ci, co, fh, fw, s) in enumerate(CONVS):
        d = inputs.conv_general(640 + i, n, h, w, ci, co, fh, fw)
        d["bias"] *= 30
        where = "conv %r pad=%d" % (CONVS[i], pad)
        if half:
            d = {key: v.astype(np.float16) for key, v in d.items()}
            got = host(tfx.tfx_conv2d_f16(dev16(d["x"]), dev16(d["filter"]), dev16(d["bias"]), s, pad, oracle.ACT_RELU6))
            assert_close_f16(got, oracle.conv2d_f16(d["x"], d["filter"], d["bias"], s, pad, oracle.ACT_RELU6), where)
        else:
            got = host(tfx.tfx_conv2d(dev(d["x"]), dev(d["filter"]), dev(d["bias"]), s, pad, oracle.ACT_RELU6))
            assert_close(got, oracle.conv2d(d["x"], d["filter"], d["bias"], s, pad, oracle.ACT_RELU6), where)


@pytest.mark.parametrize("half", [False, True])
def test_nan_and_inf_beside_ragged_edges(half):
    """Values past a row's or a tap's end are read and masked: a NaN or Inf there must not reach an output it does not
    belong to."""
    import paper_1901_05350_amd as tfx
    conv, up, dt = (tfx.tfx_conv2d_f16, dev16, np.float16) if half else (tfx.tfx_conv2d, dev, np.float32)
    for ci, co, hw in ((5, 9, 6), (33, 17, 70)):
        d = inputs.conv_general(677, 2, hw, hw, ci, co, 3, 3)
        x, f = d["x"].astype(dt), d["filter"].astype(dt)
        clean = host(conv(up(x), up(f)))
        x[1, 3, 3, 0] = np.nan
        x[0, hw - 1, hw - 1, ci - 1] = np.inf
        got = host(conv(up(x), up(f)))
        touched = np.zeros(got.shape[:3], bool)
        touched[1, 2:5, 2:5] = True
        touched[0, hw - 2:, hw - 2:] = True
        assert np.array_equal(got[~touched], clean[~touched])
        assert not np.isfinite(got[touched]).any()
