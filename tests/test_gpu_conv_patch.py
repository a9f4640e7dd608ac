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
         (5, 6, 5, 64, 8, 2, 3, 1, 0), (2, 12, 17, 64, 264, 1, 4, 3, 0), (9, 2, 3, 64, 40, 2, 3, 7, 0)]      # the last: one output per image, stride beyond it


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


def conv(args, per_channel, y_fmt=None, y_scale=None, bias=None, res=None, relu=False, absmax=None, fp32=True):
    """The entry point for this form: (Y or None, codes or None)."""
    if per_channel:
        return B.dybit_conv2d_pc(*args, bias, res, relu, absmax, y_fmt, y_scale, fp32)
    if y_fmt is None:
        return B.dybit_conv2d_ex(*args, bias, res, relu, absmax), None
    return B.dybit_conv2d_wb(*args, y_fmt, y_scale, bias, res, relu, absmax, fp32=fp32)


@pytest.mark.parametrize("per_channel", [False, True])
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("x_fmt,w_fmt", [((8, True), (8, True)), ((4, True), (4, True)), ((6, True), (4, True)), ((2, True), (6, True))])
@pytest.mark.parametrize("geom", [(3, 7, 7, 128, 208, 3, 3, 1, 1), (2, 13, 11, 64, 48, 3, 3, 2, 1)])
def test_signs_scales_and_both_outputs(patch, geom, x_fmt, w_fmt, relu, per_channel):
    """Results of both signs as signed codes, a weight scale per output channel, fp32 results and codes with either form of shortcut."""
    Bn, H, W, Cin, Cout, kh, kw, stride, pad = geom
    rng = np.random.default_rng(Cout + 2 * relu + per_channel)
    qx, qw = random_codes(rng, (Bn, H, W, Cin), x_fmt), random_codes(rng, (Cout, kh, kw, Cin), w_fmt)
    bias, sw = rng.normal(0, 1, Cout).astype(np.float32), rng.uniform(0.004, 0.2, Cout).astype(np.float32) if per_channel else np.float32(0.05)
    Ho, Wo = (H + 2 * pad - kh) // stride + 1, (W + 2 * pad - kw) // stride + 1
    want, den = R.conv2d(qx, x_fmt, 0.21, qw, w_fmt, sw, stride, pad, bias, relu)
    args = (*geom, pack_rows_dev(qx.reshape(-1, Cin), x_fmt[0]), x_fmt, scalar(0.21), pack_rows_dev(qw.reshape(Cout, -1), w_fmt[0]), w_fmt,
            dev(sw) if per_channel else scalar(sw))
    name = "f8_patch" if x_fmt[0] <= 4 and w_fmt[0] <= 4 else "f16_patch"
    mx = torch.zeros(5, dtype=torch.float32, device="cuda")
    y, _ = conv(args, per_channel, bias=dev(bias), relu=relu, absmax=mx[0:1])
    assert B.dybit_last_gemm_kernel() == name
    got = y.cpu().numpy()
    assert_within(got, want, den)
    assert relu or (got < 0).mean() > 0.2                                       # signs are really there
    assert mx[0].item() == np.abs(got).max()
    res = dev(rng.normal(0, 3, got.shape).astype(np.float32))
    r_fmt, rs = (4, True), scalar(0.7)
    rc = pack_rows_dev(random_codes(rng, (Bn * Ho * Wo, Cout), r_fmt), r_fmt[0])
    short = B.dybit_dequantize(rc, Bn * Ho * Wo * Cout, rs, *r_fmt).reshape(got.shape)
    y_res, _ = conv(args, per_channel, bias=dev(bias), res=res, relu=relu)
    y_short, _ = conv(args, per_channel, bias=dev(bias), res=short, relu=relu)
    for y_fmt in ((4, True), (6, True), (8, True)):
        s = np.float32(np.abs(got).max() * 0.7 / R.vmax(*y_fmt))
        codes_of = lambda t: R.pack_rows(R.quantize(t.cpu().numpy().reshape(-1, Cout), s, *y_fmt), y_fmt[0]).ravel()   # noqa: E731
        for fp32 in (False, True):
            z, codes = conv(args, per_channel, y_fmt, scalar(s), dev(bias), None, relu, mx[1:2].zero_(), fp32)
            assert B.dybit_last_gemm_kernel() == name
            assert np.array_equal(codes.cpu().numpy().ravel(), codes_of(y)) and mx[0].item() == mx[1].item()
            assert z is None or torch.equal(z, y)
        z, codes = conv(args, per_channel, y_fmt, scalar(s), dev(bias), res, relu, mx[1:2].zero_())
        assert B.dybit_last_gemm_kernel() == name
        assert torch.equal(z, y_res) and np.array_equal(codes.cpu().numpy().ravel(), codes_of(y_res)) and mx[1].item() == y_res.abs().max().item()
        if per_channel:
            continue                                                            # no entry point with a coded shortcut
        for fp32 in (False, True):
            z, codes = B.dybit_conv2d_wb_rc(*args, y_fmt, scalar(s), rc, r_fmt, rs, dev(bias), relu, mx[1:2].zero_(), fp32=fp32)
            assert B.dybit_last_gemm_kernel() == name
            assert np.array_equal(codes.cpu().numpy().ravel(), codes_of(y_short)) and mx[1].item() == y_short.abs().max().item()
            assert z is None or torch.equal(z, y_short)
    assert B.dybit_get_last_async_error() == B.OK


@pytest.mark.parametrize("x_fmt,w_fmt,sa,sw,sc", [((8, False), (8, True), 2.0 ** 60, 2.0 ** 56, 2.0 ** 100), ((6, False), (6, True), 2.0 ** 60, 2.0 ** 54, 2.0 ** 100),
                                                  ((8, False), (8, True), 2.0 ** -55, 2.0 ** -35, 2.0 ** -98), ((4, False), (4, True), 2.0 ** 60, 2.0 ** 42, 2.0 ** 100)])
def test_extreme_scales(patch, x_fmt, w_fmt, sa, sw, sc):
    """Scales whose product times the weights' power of two leaves the float range (6- and 8-bit weights), while the results stay inside it."""
    rng = np.random.default_rng(7)
    qx, qw = rng.integers(0, 4, (2, 9, 8, 64)).astype(np.uint8), random_codes(rng, (40, 3, 3, 64), w_fmt)
    half = 1 << (w_fmt[0] - 1)
    qw = np.where(rng.random(qw.shape) < 0.06, (qw & half) | (qw & 3), 0).astype(np.uint8)      # few and small: the first steps of either format
    args = (2, 9, 8, 64, 40, 3, 3, 1, 1, pack_rows_dev(qx.reshape(-1, 64), x_fmt[0]), x_fmt, scalar(sa), pack_rows_dev(qw.reshape(40, -1), w_fmt[0]), w_fmt, scalar(sw))
    y = B.dybit_conv2d(*args)
    assert B.dybit_last_gemm_kernel().endswith("_patch")
    want, den = R.conv2d(qx, x_fmt, sa, qw, w_fmt, sw, 1, 1, None, False)
    assert_within(y.cpu().numpy(), want, den)
    for y_fmt in ((8, True), (4, True)):
        want_codes = R.pack_rows(R.quantize(y.cpu().numpy().reshape(-1, 40), np.float32(sc), *y_fmt), y_fmt[0]).ravel()
        assert len(np.unique(want_codes)) > 4                                   # not all saturated, not all zero
        for fp32 in (False, True):
            z, codes = B.dybit_conv2d_wb(*args, y_fmt, scalar(sc), fp32=fp32)
            assert B.dybit_last_gemm_kernel().endswith("_patch")
            assert np.array_equal(codes.cpu().numpy().ravel(), want_codes)
            assert z is None or torch.equal(z, y)
    assert B.dybit_get_last_async_error() == B.OK


@pytest.mark.parametrize("sc", [float("nan"), 0.0, -1.0, float("inf"), 2.0 ** 120])
@pytest.mark.parametrize("x_fmt,w_fmt", [((8, False), (8, True)), ((4, False), (4, True))])
@pytest.mark.parametrize("fp32", [False, True])
def test_unusable_output_scale(patch, x_fmt, w_fmt, sc, fp32):
    """No codes, and the call is flagged; the fp32 results are unaffected."""
    rng = np.random.default_rng(3)
    qx, qw = random_codes(rng, (2, 9, 8, 64), x_fmt), random_codes(rng, (40, 3, 3, 64), w_fmt)
    args = (2, 9, 8, 64, 40, 3, 3, 1, 1, pack_rows_dev(qx.reshape(-1, 64), x_fmt[0]), x_fmt, scalar(0.5), pack_rows_dev(qw.reshape(40, -1), w_fmt[0]), w_fmt, scalar(0.25))
    out = torch.full((144, 40), 7, dtype=torch.uint8, device="cuda")
    z, _ = B.dybit_conv2d_wb(*args, (8, True), scalar(sc), fp32=fp32, codes_out=out)
    assert B.dybit_last_gemm_kernel().endswith("_patch")
    torch.cuda.synchronize()
    assert B.dybit_get_last_async_error() == B.ERR_BAD_SCALE
    assert bool((out == 7).all()) and (z is None or torch.equal(z, B.dybit_conv2d(*args)))


@pytest.mark.parametrize("x_fmt,w_fmt", [((4, False), (4, True)), ((8, True), (4, True)), ((2, True), (2, True)), ((6, False), (8, True))])
@pytest.mark.parametrize("groups,cin,cout,per_channel", [(2, 128, 128, False), (3, 192, 120, True), (2, 256, 512, False)])
def test_channel_slices(patch, x_fmt, w_fmt, groups, cin, cout, per_channel):
    """One launch per group of a grouped convolution: a pixel's channels are a slice of every pixel's."""
    rng = np.random.default_rng(cin + groups)
    Bn, H, W = 2, 9, 11
    qx, qw = random_codes(rng, (Bn, H, W, cin), x_fmt), random_codes(rng, (cout, 3, 3, cin // groups), w_fmt)
    bias, res = rng.normal(0, 1, cout).astype(np.float32), rng.normal(0, 5, (Bn, H, W, cout)).astype(np.float32)
    sw = rng.uniform(0.004, 0.2, cout).astype(np.float32) if per_channel else np.float32(0.05)
    want, den = R.group_conv2d(qx, x_fmt, 0.21, qw, w_fmt, sw, 1, 1, groups, bias, True, res)
    mx = torch.zeros(1, dtype=torch.float32, device="cuda")
    y = B.dybit_group_conv2d(Bn, H, W, cin, cout, 3, 3, 1, 1, groups, pack_rows_dev(qx.reshape(-1, cin), x_fmt[0]), x_fmt, scalar(0.21),
                             pack_rows_dev(qw.reshape(cout, -1), w_fmt[0]), w_fmt, dev(sw) if per_channel else scalar(sw), bias=dev(bias), residual=dev(res),
                             relu=True, absmax=mx, per_channel=per_channel)
    assert B.dybit_last_gemm_kernel() == ("f8_patch" if x_fmt[0] <= 4 and w_fmt[0] <= 4 else "f16_patch")
    got = y.cpu().numpy()
    assert_within(got, want, den, shortcut=True)
    assert mx.item() == np.abs(got).max()


# the splits of a workgroup that only large outputs get: 4-bit values times powers of two sum up exactly, in any order
@pytest.mark.parametrize("Bn,side,cin,cout,a_bits", [(43, 56, 64, 64, 4), (43, 56, 64, 40, 8), (34, 31, 128, 256, 4), (66, 32, 64, 136, 6), (20, 7, 512, 512, 4), (20, 7, 256, 512, 8),
                                                    (20, 33, 128, 72, 4), (20, 33, 64, 72, 8), (16, 33, 128, 136, 4), (16, 33, 128, 136, 6), (7, 80, 64, 72, 4), (7, 80, 64, 72, 8)])
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


def exact_codes(gen, n, fmt):
    """n packed codes of magnitudes up to 2 on the grid of halves: sums of fewer than 2^20 products are exact in fp32, in any order."""
    book = np.abs(R.codebook(*fmt))
    codes = torch.tensor(np.flatnonzero((book <= 2) & (book * 2 == np.floor(book * 2))).astype(np.int32), device="cuda")
    q = codes[torch.randint(0, len(codes), (n,), device="cuda", generator=gen)]
    per = {2: 4, 4: 2, 6: 4, 8: 1}[fmt[0]]
    word = sum(q.view(-1, per)[:, i] << (fmt[0] * i) for i in range(per))
    return torch.stack([(word >> (8 * i)) & 255 for i in range(per * fmt[0] // 8)], 1).to(torch.uint8).reshape(-1)


#  B  side  Cin  Cout k  s  A  W -> whether it is taken unasked
@pytest.mark.parametrize("Bn,side,cin,cout,k,stride,a_bits,w_bits,takes", [
    (15, 23, 128, 64, 3, 1, 8, 4, False), (36, 16, 128, 64, 3, 1, 6, 4, True), (3, 33, 256, 64, 3, 1, 4, 4, False), (33, 15, 64, 64, 3, 1, 4, 4, True),
    (13, 56, 64, 64, 3, 1, 8, 8, True), (14, 56, 64, 64, 3, 1, 8, 8, False), (14, 56, 64, 64, 3, 1, 8, 4, True), (14, 112, 64, 64, 3, 2, 4, 4, False),
    (40, 16, 256, 256, 2, 2, 4, 4, False), (64, 28, 256, 256, 3, 1, 8, 8, False), (64, 7, 512, 512, 3, 1, 6, 6, True), (4, 14, 64, 64, 1, 1, 4, 4, False)])
def test_rule(Bn, side, cin, cout, k, stride, a_bits, w_bits, takes):
    """The line between this kernel and those it replaces, from both sides; same values on either."""
    gen = torch.Generator(device="cuda").manual_seed(side + cin)
    x, w = exact_codes(gen, Bn * side * side * cin, (a_bits, False)), exact_codes(gen, cout * k * k * cin, (w_bits, True))
    args = (Bn, side, side, cin, cout, k, k, stride, k // 2 if k != 2 else 0, x, (a_bits, False), scalar(0.5), w, (w_bits, True), scalar(0.25))
    y = B.dybit_conv2d(*args)
    assert B.dybit_last_gemm_kernel().endswith("_patch") == takes
    B.dybit_set_option("gemm_kernel", "general" if takes else "patch")
    z = B.dybit_conv2d(*args)
    ran = B.dybit_last_gemm_kernel()
    B.dybit_set_option("gemm_kernel", "auto")
    assert ran == "general" if takes else ran.endswith("_patch") == (k > 1)    # a single tap is declined, whatever is asked for
    assert torch.equal(y, z) and y.std() > 0.1
