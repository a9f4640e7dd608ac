"""Few-channel convolutions on the kernel that decodes its input once per unit of output rows, against the oracle: filter rows
of 28 and 32 codes, odd filter heights, last units of fewer rows, output widths that are no multiple of 32, several images,
groups of 64 output channels with a partial last one; fp32 results with shortcut and maximum, and codes only."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import dev, scalar, pack_rows_dev, assert_within
from test_gpu_gemm import random_codes

pytestmark = pytest.mark.gpu

#        B  H   W   Cin Cout kh kw s  p
GEOMS = [(1, 97, 103, 4, 64, 7, 7, 2, 3), (2, 64, 70, 4, 64, 9, 8, 2, 3), (3, 31, 27, 8, 70, 3, 3, 1, 1), (1, 50, 49, 16, 19, 3, 2, 1, 0),
         (5, 23, 21, 8, 150, 5, 4, 1, 2), (1, 400, 9, 4, 40, 2, 5, 2, 8)]


@pytest.fixture
def few():
    B.dybit_set_option("gemm_kernel", "few")                                    # also where another kernel is the faster one
    yield
    B.dybit_set_option("gemm_kernel", "auto")


@pytest.mark.parametrize("x_fmt,w_fmt", [((8, True), (8, True)), ((6, False), (4, True)), ((4, False), (6, True)), ((6, True), (2, True))])
@pytest.mark.parametrize("geom", GEOMS)
def test_few_channel_kernel(few, x_fmt, w_fmt, geom):
    Bn, H, W, Cin, Cout, kh, kw, stride, pad = geom
    if (kh * kw * Cin * w_fmt[0]) % 8 or (Cin * w_fmt[0]) % 8:
        pytest.skip("filters of whole bytes")
    rng = np.random.default_rng(Cin + Cout)
    qx, qw = random_codes(rng, (Bn, H, W, Cin), x_fmt), random_codes(rng, (Cout, kh, kw, Cin), w_fmt)
    bias = rng.normal(0, 1, Cout).astype(np.float32)
    Ho, Wo = (H + 2 * pad - kh) // stride + 1, (W + 2 * pad - kw) // stride + 1
    res = rng.normal(0, 3, (Bn, Ho, Wo, Cout)).astype(np.float32)
    want, den = R.conv2d(qx, x_fmt, 0.21, qw, w_fmt, 0.05, stride, pad, bias, True, res)
    args = (Bn, H, W, Cin, Cout, kh, kw, stride, pad, pack_rows_dev(qx.reshape(-1, Cin), x_fmt[0]), x_fmt, scalar(0.21),
            pack_rows_dev(qw.reshape(Cout, -1), w_fmt[0]), w_fmt, scalar(0.05))
    mx = torch.zeros(2, dtype=torch.float32, device="cuda")
    y = B.dybit_conv2d_ex(*args, dev(bias), dev(res), True, mx[0:1])
    ran = B.dybit_last_gemm_kernel()
    torch.cuda.synchronize()
    assert ran == "f16_few"
    got = y.cpu().numpy()
    assert_within(got, want, den, shortcut=True)
    assert mx[0].item() == np.abs(got).max()
    if Cout % 8:
        return
    # codes only: those of the fp32 results the same kernel writes
    y = B.dybit_conv2d_ex(*args, dev(bias), None, True, mx[0:1].zero_())
    for y_fmt in ((4, False), (8, False)):
        s = np.float32(y.max().item() * 0.8 / R.vmax(*y_fmt))
        codes = torch.full((Bn * Ho * Wo * Cout * y_fmt[0] // 8 + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        B.dybit_conv2d_wb(*args, y_fmt, scalar(s), dev(bias), None, True, mx[1:2].zero_(), fp32=False, codes_out=codes[:-64])
        assert B.dybit_last_gemm_kernel() == "f16_few"
        torch.cuda.synchronize()
        assert bool((codes[-64:] == 0xA5).all()) and mx[0].item() == mx[1].item()
        want_codes = R.pack_rows(R.quantize(y.cpu().numpy().reshape(-1, Cout), s, *y_fmt), y_fmt[0])
        assert np.array_equal(codes[:-64].cpu().numpy(), want_codes.ravel())


def test_every_tap_reaches_its_pixel():
    """A single non-zero filter code: the result is the input pixel that tap sees (zero outside the image)."""
    x_fmt, w_fmt = (8, False), (4, True)
    rng = np.random.default_rng(3)
    qx = random_codes(rng, (1, 96, 98, 4), x_fmt)
    qw = np.zeros((7 * 7, 7, 7, 4), dtype=np.uint8)
    one = int(np.argmax(R.codebook(*w_fmt) == 1.0))
    for t in range(49):
        qw[t, t // 7, t % 7, t % 4] = one
    y = B.dybit_conv2d(1, 96, 98, 4, 49, 7, 7, 2, 3, pack_rows_dev(qx.reshape(-1, 4), 8), x_fmt, scalar(1.0), pack_rows_dev(qw.reshape(49, -1), 4), w_fmt, scalar(1.0))
    assert B.dybit_last_gemm_kernel() == "f16_few"
    torch.cuda.synchronize()
    want, _ = R.conv2d(qx, x_fmt, 1.0, qw, w_fmt, 1.0, 2, 3)
    assert np.array_equal(y.cpu().numpy(), want.astype(np.float32))


def test_padding_and_stride_past_32_bits():
    """The patch of such a convolution does not fit the LDS by far (its size leaves 32 bits): another kernel takes it."""
    x_fmt, w_fmt, stride, pad = (8, False), (8, True), 1 << 26, 1 << 30
    rng = np.random.default_rng(9)
    qx, qw = random_codes(rng, (2, 8, 8, 4), x_fmt), random_codes(rng, (8, 3, 3, 4), w_fmt)
    y = B.dybit_conv2d(2, 8, 8, 4, 8, 3, 3, stride, pad, pack_rows_dev(qx.reshape(-1, 4), 8), x_fmt, scalar(0.3), pack_rows_dev(qw.reshape(8, -1), 8), w_fmt,
                       scalar(0.02))
    assert y.shape == (2, 33, 33, 8) and B.dybit_last_gemm_kernel() != "f16_few"
    want, den = R.conv2d(np.ascontiguousarray(qx[:, :3, :3]), x_fmt, 0.3, qw, w_fmt, 0.02, 1, 0)   # output (16, 16) sees the image's corner
    got = y.cpu().numpy()
    assert_within(got[:, 16:17, 16:17], want, den)
    got[:, 16, 16] = 0
    assert not got.any()


# filter, N, side of the output (no padding; stride 2 for four channels, else 1), codes out -> whether the kernel takes it unasked
@pytest.mark.parametrize("cin,kh,kw,n,side,codes,takes", [
    (4, 8, 8, 64, 240, True, False), (4, 8, 8, 64, 256, True, True), (4, 8, 8, 64, 511, False, False), (4, 8, 8, 64, 512, False, True),   # row mode takes them as well
    (4, 8, 8, 160, 512, False, False), (4, 8, 8, 160, 628, False, True), (4, 8, 8, 160, 256, True, False), (4, 8, 8, 160, 300, True, True), (16, 2, 2, 160, 512, True, False),
    (8, 5, 2, 64, 300, False, False), (8, 5, 2, 64, 320, False, True), (8, 5, 2, 96, 320, False, False), (8, 7, 4, 128, 314, False, True),  # 16 codes at a time
    (8, 2, 2, 64, 340, False, False), (8, 2, 2, 64, 363, False, True), (8, 2, 2, 64, 46, True, True), (8, 2, 2, 64, 45, True, False),
    (4, 7, 7, 64, 46, False, True), (8, 3, 3, 64, 46, False, True), (8, 3, 3, 64, 130, False, False), (8, 3, 3, 64, 203, False, True), (8, 3, 1, 64, 200, False, False),
    (8, 1, 3, 160, 222, False, True), (8, 1, 3, 64, 222, False, False)])
def test_rule(cin, kh, kw, n, side, codes, takes):
    """The line between this kernel and those it replaces, from both sides; same values on either."""
    stride = 8 // min(cin, 8)
    H, W = (side - 1) * stride + kh, (side - 1) * stride + kw
    x = torch.randint(0, 256, (H * W * cin,), dtype=torch.uint8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(side))
    w = torch.randint(0, 256, (n * kh * kw * cin,), dtype=torch.uint8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    args = (1, H, W, cin, n, kh, kw, stride, 0, x, (8, False), scalar(0.3), w, (8, True), scalar(0.02))
    call = (lambda: B.dybit_conv2d_wb(*args, (8, False), scalar(1.0), relu=True, fp32=False)[1]) if codes else (lambda: B.dybit_conv2d(*args))
    y = call()
    assert (B.dybit_last_gemm_kernel() == "f16_few") == takes
    B.dybit_set_option("gemm_kernel", "few" if not takes else "general")
    other = call()
    B.dybit_set_option("gemm_kernel", "auto")
    a, b = (t.double() if not codes else t.short().double() for t in (y, other))
    assert (a - b).abs().max() <= (1 if codes else 1e-5 * kh * kw * cin * 0.006 * 128 * 64)   # sums in another order: a code beside, 1e-5 of sum |a b|


@pytest.mark.parametrize("width,takes", [(4552, True), (4554, False)])
def test_lds_of_a_compute_unit(few, width, takes):
    """Codes out, 4 x 8 taps of 4 channels: 4 rows of 8 bytes a column, 17920 for weights and columns and 256 of the kernel's own in 160 KiB."""
    gen = torch.Generator(device="cuda").manual_seed(width)
    x, w = (torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=gen) for n in (4 * width * 4, 64 * 4 * 8 * 4))
    args = (1, 4, width, 4, 64, 4, 8, 2, 0, x, (8, False), scalar(0.3), w, (8, True), scalar(0.02), (8, False), scalar(1.0))
    _, codes = B.dybit_conv2d_wb(*args, relu=True, fp32=False)
    assert (B.dybit_last_gemm_kernel() == "f16_few") == takes
    B.dybit_set_option("gemm_kernel", "general")
    _, other = B.dybit_conv2d_wb(*args, relu=True, fp32=False)
    assert (codes.short() - other.short()).abs().max() <= 1                        # sums of 128 products in another order: a code beside
