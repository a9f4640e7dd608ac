"""Convolutions of 64 and more channels on the kernel that decodes its input once per tile of outputs, against the oracle: outputs
that are no multiple of a tile, tiles over several images, strides, filters of all shapes, columns past a wave's, both splits of K."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import dev, scalar, pack_rows_dev, assert_within
from test_gpu_gemm import random_codes

pytestmark = pytest.mark.gpu

#        B  H   W   Cin  Cout kh kw s  p
GEOMS = [(1, 14, 14, 64, 64, 3, 3, 1, 1), (3, 7, 7, 128, 200, 3, 3, 1, 1), (2, 13, 11, 192, 40, 3, 3, 2, 1), (3, 15, 12, 64, 72, 3, 3, 2, 1), (1, 9, 30, 64, 136, 5, 3, 1, 1),
         (5, 6, 5, 64, 8, 2, 3, 1, 0), (2, 12, 17, 64, 264, 1, 4, 3, 0)]


@pytest.fixture
def patch():
    B.dybit_set_option("gemm_kernel", "patch")                                  # also where another kernel is the faster one
    yield
    B.dybit_set_option("gemm_kernel", "auto")


@pytest.mark.parametrize("x_fmt,w_fmt", [((8, True), (8, True)), ((6, False), (4, True)), ((8, False), (6, True)), ((6, True), (2, True)), ((4, False), (4, True)),
                                         ((4, True), (2, True)), ((2, False), (4, True)), ((2, True), (2, True)), ((4, True), (8, True)), ((2, False), (6, True))])
@pytest.mark.parametrize("geom", GEOMS)
def test_patch_kernel(patch, x_fmt, w_fmt, geom):
    Bn, H, W, Cin, Cout, kh, kw, stride, pad = geom
    rng = np.random.default_rng(Cin + Cout)
    qx, qw = random_codes(rng, (Bn, H, W, Cin), x_fmt), random_codes(rng, (Cout, kh, kw, Cin), w_fmt)
    bias = rng.normal(0, 1, Cout).astype(np.float32)
    Ho, Wo = (H + 2 * pad - kh) // stride + 1, (W + 2 * pad - kw) // stride + 1
    res = rng.normal(0, 3, (Bn, Ho, Wo, Cout)).astype(np.float32)
    want, den = R.conv2d(qx, x_fmt, 0.21, qw, w_fmt, 0.05, stride, pad, bias, True, res)
    args = (Bn, H, W, Cin, Cout, kh, kw, stride, pad, pack_rows_dev(qx.reshape(-1, Cin), x_fmt[0]), x_fmt, scalar(0.21),
            pack_rows_dev(qw.reshape(Cout, -1), w_fmt[0]), w_fmt, scalar(0.05))
    name = "f8_patch" if x_fmt[0] <= 4 and w_fmt[0] <= 4 else "f16_patch"
    mx = torch.zeros(4, dtype=torch.float32, device="cuda")
    y = B.dybit_conv2d_ex(*args, dev(bias), dev(res), True, mx[0:1])
    ran = B.dybit_last_gemm_kernel()
    torch.cuda.synchronize()
    assert ran == name
    got = y.cpu().numpy()
    assert_within(got, want, den, shortcut=True)
    assert mx[0].item() == np.abs(got).max()
    # codes only, with and without a shortcut given as codes: those of the fp32 results the same kernel writes
    y = B.dybit_conv2d_ex(*args, dev(bias), None, True, mx[0:1].zero_())
    for y_fmt in ((4, False), (6, True), (8, False)):
        if Cout * y_fmt[0] % 32:
            continue
        s = np.float32(y.max().item() * 0.8 / R.vmax(*y_fmt))
        codes = torch.full((Bn * Ho * Wo * Cout * y_fmt[0] // 8 + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        B.dybit_conv2d_wb(*args, y_fmt, scalar(s), dev(bias), None, True, mx[1:2].zero_(), fp32=False, codes_out=codes[:-64])
        assert B.dybit_last_gemm_kernel() == name
        torch.cuda.synchronize()
        assert bool((codes[-64:] == 0xA5).all()) and mx[0].item() == mx[1].item()
        want_codes = R.pack_rows(R.quantize(y.cpu().numpy().reshape(-1, Cout), s, *y_fmt), y_fmt[0])
        assert np.array_equal(codes[:-64].cpu().numpy(), want_codes.ravel())
        both, codes = B.dybit_conv2d_wb(*args, y_fmt, scalar(s), dev(bias), None, True, mx[1:2].zero_())        # fp32 as well
        assert B.dybit_last_gemm_kernel() == name
        torch.cuda.synchronize()
        assert torch.equal(both, y) and mx[0].item() == mx[1].item() and np.array_equal(codes.cpu().numpy().ravel(), want_codes.ravel())
        r_fmt = {4: (8, False), 6: (4, True), 8: (6, False)}[y_fmt[0]]
        if Cout * r_fmt[0] % 32:
            continue
        qr = random_codes(rng, (Bn * Ho * Wo, Cout), r_fmt)
        rc, rs = pack_rows_dev(qr, r_fmt[0]), scalar(0.4)
        short = B.dybit_dequantize(rc, Bn * Ho * Wo * Cout, rs, *r_fmt).reshape(Bn, Ho, Wo, Cout)
        z = B.dybit_conv2d_ex(*args, dev(bias), short, True, mx[2:3].zero_())
        _, codes = B.dybit_conv2d_wb_rc(*args, y_fmt, scalar(s), rc, r_fmt, rs, dev(bias), True, mx[3:4].zero_(), fp32=False)
        assert B.dybit_last_gemm_kernel() == name
        torch.cuda.synchronize()
        assert mx[2].item() == mx[3].item()
        want_codes = R.pack_rows(R.quantize(z.cpu().numpy().reshape(-1, Cout), s, *y_fmt), y_fmt[0])
        assert np.array_equal(codes.cpu().numpy().ravel(), want_codes.ravel())


# the splits of a workgroup that only large outputs get: 4-bit values times powers of two sum up exactly, in any order
@pytest.mark.parametrize("Bn,side,cin,cout,a_bits", [(43, 56, 64, 64, 4), (43, 56, 64, 40, 8), (34, 31, 128, 256, 4), (66, 32, 64, 136, 6), (20, 7, 512, 512, 4), (20, 7, 256, 512, 8)])
def test_splits_agree_with_the_general_kernel(patch, Bn, side, cin, cout, a_bits):
    gen = torch.Generator(device="cuda").manual_seed(cin + cout)
    x = torch.randint(0, 256, (Bn * side * side * cin * a_bits // 8,), dtype=torch.uint8, device="cuda", generator=gen)
    w = torch.randint(0, 256, (cout * 9 * cin // 2,), dtype=torch.uint8, device="cuda", generator=gen)
    args = (Bn, side, side, cin, cout, 3, 3, 1, 1, x, (a_bits, False), scalar(0.5), w, (4, True), scalar(0.25))
    bias = torch.randint(-9, 9, (cout,), device="cuda", generator=gen).float()
    y = B.dybit_conv2d_ex(*args, bias, None, True)
    assert B.dybit_last_gemm_kernel().endswith("_patch")
    _, codes = B.dybit_conv2d_wb(*args, (4, False), scalar(64.0), bias, None, True, fp32=False)
    assert B.dybit_last_gemm_kernel().endswith("_patch")
    B.dybit_set_option("gemm_kernel", "general")
    assert torch.equal(y, B.dybit_conv2d_ex(*args, bias, None, True))
    _, other = B.dybit_conv2d_wb(*args, (4, False), scalar(64.0), bias, None, True, fp32=False)
    assert torch.equal(codes, other)


@pytest.mark.parametrize("width,takes", [(495, True), (496, False)])
def test_lds_of_a_compute_unit(patch, width, takes):
    """Codes out of 8-bit operands: 130 + 2 W + 1 pixels of 144 bytes, 2064 for the columns and 256 of the kernel's own in 160 KiB."""
    gen = torch.Generator(device="cuda").manual_seed(width)
    x, w = (torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=gen) for n in (3 * width * 64, 64 * 9 * 64))
    args = (1, 3, width, 64, 64, 3, 3, 1, 1, x, (8, False), scalar(0.5), w, (8, True), scalar(0.25), (8, False), scalar(64.0))
    _, codes = B.dybit_conv2d_wb(*args, relu=True, fp32=False)
    assert (B.dybit_last_gemm_kernel() == "f16_patch") == takes
    B.dybit_set_option("gemm_kernel", "general")
    _, other = B.dybit_conv2d_wb(*args, relu=True, fp32=False)
    # 576 products in fp32, in another order: within 576 2^-24 of their sum, so a code apart at most
    assert (codes.short() - other.short()).abs().max() <= 1


#  B  side  Cin  Cout k  s  A  W -> whether it is taken unasked
@pytest.mark.parametrize("Bn,side,cin,cout,k,stride,a_bits,w_bits,takes", [
    (15, 23, 128, 64, 3, 1, 8, 4, False), (36, 16, 128, 64, 3, 1, 6, 4, True), (3, 33, 256, 64, 3, 1, 4, 4, False), (33, 15, 64, 64, 3, 1, 4, 4, True),
    (13, 56, 64, 64, 3, 1, 8, 8, True), (14, 56, 64, 64, 3, 1, 8, 8, False), (14, 56, 64, 64, 3, 1, 8, 4, True), (14, 112, 64, 64, 3, 2, 4, 4, False),
    (40, 16, 256, 256, 2, 2, 4, 4, False), (64, 28, 256, 256, 3, 1, 8, 8, False), (64, 7, 512, 512, 3, 1, 6, 6, True), (4, 14, 64, 64, 1, 1, 4, 4, False)])
def test_rule(Bn, side, cin, cout, k, stride, a_bits, w_bits, takes):
    """The line between this kernel and those it replaces, from both sides; same values on either."""
    gen = torch.Generator(device="cuda").manual_seed(side + cin)
    x = torch.randint(0, 256, (Bn * side * side * cin * a_bits // 8,), dtype=torch.uint8, device="cuda", generator=gen)
    w = torch.randint(0, 256, (cout * k * k * cin * w_bits // 8,), dtype=torch.uint8, device="cuda", generator=gen)
    args = (Bn, side, side, cin, cout, k, k, stride, k // 2 if k != 2 else 0, x, (a_bits, False), scalar(0.5), w, (w_bits, True), scalar(0.25))
    y = B.dybit_conv2d(*args)
    assert B.dybit_last_gemm_kernel().endswith("_patch") == takes
    B.dybit_set_option("gemm_kernel", "general" if takes else "patch")
    z = B.dybit_conv2d(*args)
    B.dybit_set_option("gemm_kernel", "auto")
    # sums of k k Cin products in fp32, in another order: K 2^-24 of the sum of their magnitudes, at most 2^(a + w - 3) / 8 each
    assert (y - z).abs().max() <= cin * k * k * 2.0 ** -24 * cin * k * k * 2.0 ** (a_bits + w_bits - 3) / 8
