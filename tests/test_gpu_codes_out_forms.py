"""Forms of the write-back whose kernel builds no other test reaches: rows that start at any byte (K no multiple of 64) with codes
out, 128 x 128 fp16 tiles in two k-groups and weight-stationary kernels of four column blocks on codes alone, one scale per
column, and the few-channel convolution with a coded shortcut, signed and 6-bit codes, and at the sizes where it takes over
filters that the weight-stationary kernel's row mode takes as well.

Each time: fp32 results against the oracle, their codes bit for bit the oracle's encoding of them, and codes alone the same codes."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import dev, scalar, pack_rows_dev, assert_within
from test_gpu_codes_only import both
from test_gpu_gemm import random_codes
from test_gpu_small_ragged import kernel  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def check_codes(got32, codes, scale, fmt):
    want = R.pack_rows(R.quantize(got32.reshape(-1, got32.shape[-1]), np.float32(scale), *fmt), fmt[0])
    assert np.array_equal(codes.cpu().numpy().reshape(want.shape), want)


@pytest.mark.parametrize("a_fmt,w_fmt", [((8, False), (4, True)), ((6, True), (6, True)), ((4, False), (4, True))])
@pytest.mark.parametrize("c_fmt,r_fmt", [((4, False), None), ((8, True), (8, True)), ((6, True), (4, False))])
@pytest.mark.parametrize("K", [68, 132, 196, 1148])
def test_rows_at_any_byte(kernel, a_fmt, w_fmt, c_fmt, r_fmt, K):
    M, N = 161, 80
    rng = np.random.default_rng(K + c_fmt[0])
    qa, qw = random_codes(rng, (M, K), a_fmt), random_codes(rng, (N, K), w_fmt)
    bias = rng.normal(0, 3, N).astype(np.float32)
    relu, kw, res = not c_fmt[1], {}, None
    if r_fmt is not None:
        qr = random_codes(rng, (M, N), r_fmt)
        kw = {"r_codes": pack_rows_dev(qr, r_fmt[0]), "r_fmt": r_fmt, "r_scale": scalar(0.03)}
        res = (R.codebook(*r_fmt)[qr].astype(np.float32) * np.float32(0.03)).astype(np.float32)
    want, den = R.gemm(qa, a_fmt, 0.37, qw, w_fmt, 0.011, bias, relu, res)
    s = np.float32(0.6 * np.abs(want).max() / R.vmax(*c_fmt))
    args = (M, N, K, pack_rows_dev(qa, a_fmt[0]), a_fmt, scalar(0.37), pack_rows_dev(qw, w_fmt[0]), w_fmt, scalar(0.011), c_fmt, scalar(s))
    c = both(args, {"bias": dev(bias), "relu": relu}, **kw).cpu().numpy()
    assert B.dybit_last_gemm_kernel() != "general"
    assert_within(c, want, den, shortcut=True)
    _, codes = (B.dybit_gemm_wb_rc if kw else B.dybit_gemm_wb)(*args, bias=dev(bias), relu=relu, **kw)
    check_codes(c, codes, s, c_fmt)


@pytest.mark.parametrize("option,a_fmt,w_fmt,N,K,ran", [("mid", (8, False), (4, True), 208, 256, "f16_128_kg2"), ("mid", (8, True), (8, True), 96, 128, "f16_128_kg2"),
                                                        ("ws", (8, False), (8, True), 96, 256, "f16_ws"), ("ws", (6, True), (4, True), 128, 192, "f16_ws")])
@pytest.mark.parametrize("c_fmt", [(4, False), (4, True), (6, False), (8, True)])
@pytest.mark.parametrize("per_channel", [False, True])
def test_codes_alone(option, a_fmt, w_fmt, N, K, ran, c_fmt, per_channel):
    M = 290
    rng = np.random.default_rng(N + K)
    qa, qw = random_codes(rng, (M, K), a_fmt), random_codes(rng, (N, K), w_fmt)
    bias = rng.normal(0, 1, N).astype(np.float32)
    sw = (rng.uniform(0.2, 5.0, N) * 0.011).astype(np.float32) if per_channel else np.float32([0.011])
    relu = not c_fmt[1]
    want, den = R.gemm(qa, a_fmt, 1.0, qw, w_fmt, 1.0)
    alpha = np.float64(np.float32(0.37)) * sw.astype(np.float64)
    want, den = want * alpha + bias, den * alpha + np.abs(bias)
    want = np.maximum(want, 0) if relu else want
    s = np.float32(0.6 * np.abs(want).max() / R.vmax(*c_fmt))
    B.dybit_set_option("gemm_kernel", option)
    B.dybit_set_option("mid_kgroups", "2" if option == "mid" else "auto")
    try:
        args = (M, N, K, pack_rows_dev(qa, a_fmt[0]), a_fmt, scalar(0.37), pack_rows_dev(qw, w_fmt[0]), w_fmt, dev(sw))
        mx = torch.zeros(2, dtype=torch.float32, device="cuda")
        tail = dict(bias=dev(bias), relu=relu, c_fmt=c_fmt, c_scale=scalar(s))
        call = B.dybit_gemm_pc if per_channel else lambda *a, c_fmt, c_scale, **k: B.dybit_gemm_wb(*a, c_fmt, c_scale, **k)
        c, codes = call(*args, absmax=mx[0:1], **tail)
        assert B.dybit_last_gemm_kernel() == ran
        none, only = call(*args, absmax=mx[1:2], fp32=False, **tail)
        assert B.dybit_last_gemm_kernel() == ran
    finally:
        B.dybit_set_option("gemm_kernel", "auto")
        B.dybit_set_option("mid_kgroups", "auto")
    torch.cuda.synchronize()
    got = c.cpu().numpy()
    assert_within(got, want, den)
    check_codes(got, codes, s, c_fmt)
    assert none is None and torch.equal(only.reshape(-1), codes.reshape(-1)) and mx[0].item() == mx[1].item()


#        B  H   W   Cin Cout kh kw s  p   sa      (the last: factors that leave the float range with the accumulators' power of two)
FEW = [(2, 64, 71, 4, 64, 7, 7, 2, 3, 0.21), (1, 61, 75, 8, 72, 3, 3, 1, 1, 0.21), (1, 101, 95, 4, 40, 7, 7, 2, 3, 2.0 ** 60),
       (4, 258, 270, 4, 32, 8, 8, 2, 3, 0.21), (4, 257, 261, 8, 40, 2, 4, 1, 0, 0.21)]


@pytest.mark.parametrize("x_fmt,w_fmt", [((8, True), (8, True)), ((6, False), (4, True))])
@pytest.mark.parametrize("y_fmt,r_fmt", [((6, False), (4, False)), ((4, True), (8, True)), ((6, True), None), ((8, True), (6, True))])
@pytest.mark.parametrize("geom", FEW)
def test_few_channels(geom, x_fmt, w_fmt, y_fmt, r_fmt):
    Bn, H, W, Cin, Cout, kh, kw, stride, pad, sa = geom
    sw = 0.05 if sa < 1 else 2.0 ** 45
    rng = np.random.default_rng(Cout + kh)
    Ho, Wo = (H + 2 * pad - kh) // stride + 1, (W + 2 * pad - kw) // stride + 1
    if (Cout * y_fmt[0]) % 32 or (r_fmt and (Cout * r_fmt[0]) % 32):
        pytest.skip("rows of codes are whole words")
    qx, qw = random_codes(rng, (Bn, H, W, Cin), x_fmt), random_codes(rng, (Cout, kh, kw, Cin), w_fmt)
    relu, bias = not y_fmt[1], (rng.normal(0, 1, Cout) * (sa * sw / 0.01)).astype(np.float32)
    want, den = R.conv2d(qx, x_fmt, sa, qw, w_fmt, sw, stride, pad, bias, False)
    s = np.float32(min(np.abs(want).max() * 0.7 / R.vmax(*y_fmt), 2.0 ** 99))
    args = (Bn, H, W, Cin, Cout, kh, kw, stride, pad, pack_rows_dev(qx.reshape(-1, Cin), x_fmt[0]), x_fmt, scalar(sa),
            pack_rows_dev(qw.reshape(Cout, -1), w_fmt[0]), w_fmt, scalar(sw), y_fmt, scalar(s))
    mx = torch.zeros(1, dtype=torch.float32, device="cuda")
    if r_fmt is None:
        _, codes = B.dybit_conv2d_wb(*args, dev(bias), None, relu, mx, fp32=False)
    else:
        qr, sr = random_codes(rng, (Bn, Ho, Wo, Cout), r_fmt), np.float32(s * R.vmax(*y_fmt) / R.vmax(*r_fmt) * 0.3)
        _, codes = B.dybit_conv2d_wb_rc(*args, pack_rows_dev(qr.reshape(-1, Cout), r_fmt[0]), r_fmt, scalar(sr), dev(bias), relu, mx, fp32=False)
        want = want + (R.codebook(*r_fmt)[qr].astype(np.float32) * sr).astype(np.float64)
    assert B.dybit_last_gemm_kernel() == "f16_few"
    want = np.maximum(want, 0) if relu else want
    torch.cuda.synchronize()
    assert B.dybit_get_last_async_error() == B.OK
    # the kernel's fp32 result lies within the product tolerance of `want`, so its code lies between those of the two ends
    tol = 1e-5 * den + 2.0 ** -23 * np.abs(want)
    assert abs(mx.item() - np.abs(want).max()) <= tol.max()
    values = R.codebook(*y_fmt)
    lo, hi = (values[R.quantize((want + d).astype(np.float32), s, *y_fmt)] for d in (-tol, tol))
    q = np.unpackbits(codes.cpu().numpy().reshape(Bn * Ho * Wo, -1), axis=1, bitorder="little").reshape(Bn, Ho, Wo, Cout, y_fmt[0])
    got = values[(q.astype(np.int64) << np.arange(y_fmt[0])).sum(-1)]
    assert ((lo <= got) & (got <= hi)).all()
    assert (lo != hi).mean() < 0.01                                              # and hardly any code is open
