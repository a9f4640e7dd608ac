"""Grouped convolutions of 64 and more channels per group: the tiled kernels on a channel slice of every pixel (forced, since the
one-launch kernel takes most such layers), the line from which they take pairs of 4- and 2-bit formats, and equal results on both
sides of it."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import dev, scalar, pack_rows_dev, assert_within
from test_gpu_gemm import random_codes

pytestmark = pytest.mark.gpu


def group_conv(shape, k, groups, qx, x_fmt, qw, w_fmt, **kw):
    Bn, H, W, cin, cout = shape
    return B.dybit_group_conv2d(Bn, H, W, cin, cout, k, k, 1, k // 2, groups, qx, x_fmt, scalar(0.21), qw, w_fmt, scalar(0.05), **kw)


@pytest.mark.parametrize("force,ran", [("mid", ("f16_128_kg1", "f16_128_kg2", "f8_128_kg1", "f8_128_kg2", "f8_64")), ("ws", ("f16_ws", "f8_ws")),
                                       ("small", ("f16_small", "f8_small")), ("large", ("f16_256", "f8_256"))])
@pytest.mark.parametrize("x_fmt,w_fmt", [((4, False), (4, True)), ((8, True), (4, True)), ((2, True), (2, True))])
@pytest.mark.parametrize("groups,cin,cout,k", [(2, 128, 128, 3), (3, 192, 120, 1), (2, 256, 512, 1)])
def test_tiled_kernels_on_channel_slices(force, ran, x_fmt, w_fmt, groups, cin, cout, k):
    rng = np.random.default_rng(cin + k)
    Bn, H, W = 2, 9, 11
    qx, qw = random_codes(rng, (Bn, H, W, cin), x_fmt), random_codes(rng, (cout, k, k, cin // groups), w_fmt)
    bias = rng.normal(0, 1, cout).astype(np.float32)
    res = rng.normal(0, 5, (Bn, H, W, cout)).astype(np.float32)
    want, den = R.group_conv2d(qx, x_fmt, 0.21, qw, w_fmt, 0.05, 1, k // 2, groups, bias, True, res)
    mx = torch.zeros(1, dtype=torch.float32, device="cuda")
    B.dybit_set_option("gemm_kernel", force)
    y = group_conv((Bn, H, W, cin, cout), k, groups, pack_rows_dev(qx.reshape(-1, cin), x_fmt[0]), x_fmt, pack_rows_dev(qw.reshape(cout, -1), w_fmt[0]), w_fmt,
                   bias=dev(bias), residual=dev(res), relu=True, absmax=mx)
    kernel = B.dybit_last_gemm_kernel()
    B.dybit_set_option("gemm_kernel", "auto")
    assert kernel in ran or (force == "large" and kernel.startswith("f16_128"))   # 2-bit fp16 operands want 128 channels there
    got = y.cpu().numpy()
    assert_within(got, want, den, shortcut=True)
    assert mx.item() == np.abs(got).max()


@pytest.mark.parametrize("x_fmt,w_fmt,geom,one", [
    ((4, False), (4, True), (16, 56, 128, 128, 3, 2), False), ((4, False), (4, True), (4, 56, 128, 128, 3, 2), True),     # outputs
    ((8, False), (4, True), (16, 56, 128, 128, 3, 2), True), ((2, False), (4, True), (32, 56, 64, 64, 3, 2), True),       # formats; weights
    ((4, False), (4, True), (16, 56, 128, 32, 3, 2), True), ((4, False), (4, True), (16, 56, 96, 128, 3, 2), True),       # columns; channels
    ((4, True), (2, True), (32, 28, 512, 512, 1, 2), False)])
def test_line(x_fmt, w_fmt, geom, one):
    Bn, hw, cg, cog, k, groups = geom
    gen = torch.Generator(device="cuda").manual_seed(hw)
    codes = lambda n, bits: torch.randint(0, 256, (n * bits // 8,), dtype=torch.uint8, device="cuda", generator=gen)   # noqa: E731
    x, w = codes(Bn * hw * hw * cg * groups, x_fmt[0]), codes(cog * groups * k * k * cg, w_fmt[0])
    shape = (Bn, hw, hw, cg * groups, cog * groups)
    y = group_conv(shape, k, groups, x, x_fmt, w, w_fmt)
    assert (B.dybit_last_gemm_kernel() == "f16_group") == one
    B.dybit_set_option("gemm_kernel", "general")
    other = group_conv(shape, k, groups, x, x_fmt, w, w_fmt)
    B.dybit_set_option("gemm_kernel", "auto")
    den = 0.21 * 0.05 * (1 << R.magnitude_bits(*x_fmt)) * (1 << R.magnitude_bits(*w_fmt)) / 4 * cg * k * k          # the largest sum |a b|
    assert (y.double() - other.double()).abs().max() <= 2e-5 * den
