"""The 3 x 3 depthwise kernel (codes read by the threads themselves, fp16 window and taps): every pair of formats at both
strides against the oracle, its write-back codes against the oracle's encoding, and the grid rule's two limits.

Tolerance: the products are exact in fp32 and the nine additions the only roundings, as in test_gpu_dwconv."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import assert_within, dev, oracle_codes, pack_rows_dev, scalar
from test_gpu_gemm import random_codes

pytestmark = pytest.mark.gpu
FMTS = [(b, s) for b in (2, 4, 8) for s in (False, True)]


@pytest.mark.parametrize("x_fmt", FMTS)
@pytest.mark.parametrize("w_fmt", FMTS)
@pytest.mark.parametrize("stride", [1, 2])
def test_every_pair_of_formats(x_fmt, w_fmt, stride):
    """Width no multiple of a thread's columns, several strips of rows with a ragged last one, images that share a workgroup."""
    rng = np.random.default_rng(x_fmt[0] * 16 + w_fmt[0])
    Bn, H, W, C = 3, 37, 22, 16
    qx, qw = random_codes(rng, (Bn, H, W, C), x_fmt), random_codes(rng, (3, 3, C), w_fmt)
    bias = rng.normal(0, 1, C).astype(np.float32)
    sw = rng.uniform(0.01, 0.1, C).astype(np.float32)
    y_fmt = (4, True) if stride == 1 else (8, False)
    mx = torch.zeros(1, dtype=torch.float32, device="cuda")
    y, codes = B.dybit_dwconv2d_wb(Bn, H, W, C, 3, 3, stride, 1, pack_rows_dev(qx.reshape(-1, C), x_fmt[0]), x_fmt, scalar(0.3),
                                   pack_rows_dev(qw.reshape(-1, C), w_fmt[0]), w_fmt, dev(sw), dev(bias), stride == 2, mx,
                                   y_fmt, scalar(0.0437), per_channel=True)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    want, den = R.dwconv2d(qx, x_fmt, 1.0, qw, w_fmt, 1.0, stride, 1)          # scales are applied to the exact sums
    alpha = 0.3 * sw.astype(np.float64)
    want, den = want * alpha + bias, den * alpha + np.abs(bias)
    if stride == 2:
        want = np.maximum(want, 0.0)
    assert_within(got, want, den)
    assert mx.item() == np.abs(got).max()
    q = R.quantize(got.reshape(-1, C), np.float32(0.0437), *y_fmt)
    assert torch.equal(codes.reshape(-1), pack_rows_dev(np.asarray(q).reshape(-1, C), y_fmt[0]).reshape(-1))
    # codes alone are the same codes
    _, only = B.dybit_dwconv2d_wb(Bn, H, W, C, 3, 3, stride, 1, pack_rows_dev(qx.reshape(-1, C), x_fmt[0]), x_fmt, scalar(0.3),
                                  pack_rows_dev(qw.reshape(-1, C), w_fmt[0]), w_fmt, dev(sw), dev(bias), stride == 2, None,
                                  y_fmt, scalar(0.0437), per_channel=True, fp32=False)
    assert torch.equal(only, codes)


def _conv(x, shape, w, C, stride=2):
    Bn, H, W = shape
    return B.dybit_dwconv2d(Bn, H, W, C, 3, 3, stride, 1, x, (8, False), scalar(0.3), w, (8, True), scalar(0.1))


def test_images_past_the_first_grid_row():
    """A batch of 2^30 bytes and more is several rows of the grid: an image of the second row gives what it gives alone."""
    n, H, W, C = 34, 1024, 1024, 32
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randint(0, 256, (n, H * W * C), dtype=torch.uint8, device="cuda", generator=g)
    w = torch.randint(0, 256, (9 * C,), dtype=torch.uint8, device="cuda", generator=g)
    y = _conv(x.reshape(-1), (n, H, W), w, C)
    for i in (0, 30, 31, 32, 33):
        assert torch.equal(y[i], _conv(x[i].clone(), (1, H, W), w, C)[0])


@pytest.mark.parametrize("stride", [1, 2])
def test_image_of_2_30_bytes(stride):
    """Such an image goes in bands of output rows, a launch each: every row is what a slice of the image gives."""
    H, W, C = 8192, 8192, 16
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randint(0, 256, (H, W * C), dtype=torch.uint8, device="cuda", generator=g)
    w = torch.randint(0, 256, (9 * C,), dtype=torch.uint8, device="cuda", generator=g)
    y = _conv(x.reshape(-1), (1, H, W), w, C, stride)[0]
    n = 1024                                                                   # input rows of a slice, two more on either side
    for r0 in range(0, H, n):
        lo, hi = max(r0 - 2, 0), min(r0 + n + 2, H)
        part = _conv(x[lo:hi].clone().reshape(-1), (1, hi - lo, W), w, C, stride)[0]
        first = (r0 - lo) // stride
        assert torch.equal(y[r0 // stride:(r0 + n) // stride], part[first:first + n // stride])
