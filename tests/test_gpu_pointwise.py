"""1 x 1 convolutions at stride 1 run as products: against the oracle's convolution for every way the channels can end (whole K
steps, whole runs, odd ones), and bit-equal to the product of the same matrices, which takes the same kernel."""
import numpy as np
import pytest

from oracle import dybit_ref as R
from gpu_util import assert_within, dev, pack_rows_dev, scalar
from paper_2302_12510_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a_fmt,w_fmt", [((4, False), (4, True)), ((8, False), (6, True)), ((6, True), (8, True)), ((2, False), (4, True))])
@pytest.mark.parametrize("cin,cout", [(4, 8), (24, 40), (64, 64), (80, 144), (128, 200), (100, 36), (320, 96)])
@pytest.mark.parametrize("Bn,H,W", [(1, 1, 1), (2, 7, 5), (3, 33, 20)])
def test_against_oracle_and_product(a_fmt, w_fmt, cin, cout, Bn, H, W):
    rng = np.random.default_rng(cin + cout + H)
    qx = rng.integers(0, 1 << a_fmt[0], (Bn, H, W, cin)).astype(np.uint8)
    qw = rng.integers(0, 1 << w_fmt[0], (cout, 1, 1, cin)).astype(np.uint8)
    bias = rng.normal(0, 1, cout).astype(np.float32)
    x, w = pack_rows_dev(qx, a_fmt[0]), pack_rows_dev(qw, w_fmt[0])
    got = B.dybit_conv2d(Bn, H, W, cin, cout, 1, 1, 1, 0, x, a_fmt, scalar(0.37), w, w_fmt, scalar(0.011), dev(bias), True)
    ran = B.dybit_last_gemm_kernel()
    want, den = R.conv2d(qx, a_fmt, 0.37, qw, w_fmt, 0.011, 1, 0, bias, True)
    assert_within(got.cpu().numpy().reshape(-1, cout), np.asarray(want).reshape(-1, cout), np.asarray(den).reshape(-1, cout))
    same = B.dybit_gemm(Bn * H * W, cout, cin, x, a_fmt, scalar(0.37), w, w_fmt, scalar(0.011), dev(bias), True)
    assert B.dybit_last_gemm_kernel() == ran
    assert np.array_equal(got.cpu().numpy().reshape(-1, cout), same.cpu().numpy())


def test_other_geometries_stay_convolutions():
    """Stride, padding or a group of a wider image: the image is not the matrix."""
    fmt, wf = (4, False), (4, True)
    rng = np.random.default_rng(2)
    qx, qw = rng.integers(0, 16, (2, 9, 8, 64)).astype(np.uint8), rng.integers(0, 16, (64, 1, 1, 64)).astype(np.uint8)
    x, w = pack_rows_dev(qx, 4), pack_rows_dev(qw, 4)
    for stride, pad in ((2, 0), (1, 1)):
        got = B.dybit_conv2d(2, 9, 8, 64, 64, 1, 1, stride, pad, x, fmt, scalar(1.0), w, wf, scalar(1.0)).cpu().numpy()
        want, den = R.conv2d(qx, fmt, 1.0, qw, wf, 1.0, stride, pad)
        assert_within(got, np.asarray(want).reshape(got.shape), np.asarray(den).reshape(got.shape))
    got = B.dybit_group_conv2d(2, 9, 8, 64, 64, 1, 1, 1, 0, 2, x, fmt, scalar(1.0), pack_rows_dev(qw[..., :32], 4), wf, scalar(1.0)).cpu().numpy()
    for i in range(2):
        want, den = R.conv2d(qx[..., 32 * i:32 * i + 32], fmt, 1.0, qw[32 * i:32 * i + 32, :, :, :32], wf, 1.0, 1, 0)
        part = got[..., 32 * i:32 * i + 32]
        assert_within(part, np.asarray(want).reshape(part.shape), np.asarray(den).reshape(part.shape))
