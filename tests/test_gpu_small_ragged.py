"""Matrix products on the small-output kernel (32-row tiles, K split over the waves of a workgroup) and products whose K is not
a multiple of 64 (rows of codes that start at any byte) on it and on the 128 x 128 kernel, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import dev, scalar, pack_rows_dev, assert_within
from test_gpu_gemm import random_codes

pytestmark = pytest.mark.gpu

PAIRS = [((4, False), (4, True)), ((2, True), (4, True)), ((8, True), (4, True)), ((8, False), (8, True)), ((6, True), (6, True)), ((4, False), (2, True)), ((2, True), (8, True)),
         ((4, True), (6, True)), ((6, False), (4, True)), ((2, False), (2, True))]
# K: one step; an odd part of 4 codes; one code group short of a step; odd parts of every k-group; more steps than waves
SHAPES = [(1, 7, 64), (33, 70, 68), (32, 32, 124), (65, 33, 128), (5, 129, 132), (130, 65, 196), (31, 257, 1148), (290, 130, 1216)]


@pytest.fixture(params=["small", "small-e4m3", "mid1", "mid2", "auto"])
def kernel(request):
    name = request.param
    B.dybit_set_option("gemm_kernel", name[:3] if name.startswith("mid") else name.split("-")[0])
    B.dybit_set_option("mid_kgroups", name[3:] or "auto" if name.startswith("mid") else "auto")
    B.dybit_set_option("gemm_mfma", "auto" if name == "small-e4m3" else "f16")
    yield name
    for k in ("gemm_kernel", "mid_kgroups", "gemm_mfma"):
        B.dybit_set_option(k, "auto")


@pytest.mark.parametrize("a_fmt,w_fmt", PAIRS)
@pytest.mark.parametrize("shape", SHAPES)
def test_products(kernel, a_fmt, w_fmt, shape):
    M, N, K = shape
    rng = np.random.default_rng(M * 7 + K)
    qa, qw = random_codes(rng, (M, K), a_fmt), random_codes(rng, (N, K), w_fmt)
    bias = rng.normal(0, 3, N).astype(np.float32)
    res = rng.normal(0, 5, (M, N)).astype(np.float32)
    want, den = R.gemm(qa, a_fmt, 0.37, qw, w_fmt, 0.011, bias, True, res)
    mx = torch.zeros(1, dtype=torch.float32, device="cuda")
    c = B.dybit_gemm_ex(M, N, K, pack_rows_dev(qa, a_fmt[0]), a_fmt, scalar(0.37), pack_rows_dev(qw, w_fmt[0]), w_fmt, scalar(0.011),
                        dev(bias), dev(res), True, mx)
    ran = B.dybit_last_gemm_kernel()
    torch.cuda.synchronize()
    low = a_fmt[0] <= 4 and w_fmt[0] <= 4
    assert ran == {"small": "f16_small", "small-e4m3": "f8_small" if low else "f16_small", "mid1": "f16_128_kg1", "auto": "f16_small",
                   "mid2": "f16_128_kg1" if K % 64 and K < 128 else "f16_128_kg2"}[kernel]
    got = c.cpu().numpy()
    assert_within(got, want, den, shortcut=True)
    assert mx.item() == np.abs(got).max()


@pytest.mark.parametrize("a_fmt,w_fmt", [((8, False), (4, True)), ((6, True), (6, True)), ((4, False), (4, True))])
@pytest.mark.parametrize("K", [128, 196])
def test_every_k_counts_once(kernel, a_fmt, w_fmt, K):
    """A single non-zero code at each k in turn: its product and nothing else (the codes beside the row must not leak in)."""
    one_a, one_w = int(np.argmax(R.codebook(*a_fmt) == 1.0)), int(np.argmax(R.codebook(*w_fmt) == 1.0))
    qa = np.full((K, K), (1 << a_fmt[0]) - 2, dtype=np.uint8)              # row i: a one at k = i and large values elsewhere
    qa[np.arange(K), np.arange(K)] = one_a
    qw = np.zeros((K, K), dtype=np.uint8)
    qw[np.arange(K), np.arange(K)] = one_w
    c = B.dybit_gemm(K, K, K, pack_rows_dev(qa, a_fmt[0]), a_fmt, scalar(1.0), pack_rows_dev(qw, w_fmt[0]), w_fmt, scalar(1.0))
    torch.cuda.synchronize()
    assert np.array_equal(c.cpu().numpy(), R.codebook(*a_fmt)[qa].astype(np.float32))


@pytest.mark.parametrize("geom", [(1, 7, 7, 128, 96, 3, 1, 1), (2, 9, 6, 64, 40, 3, 2, 1), (3, 5, 5, 192, 64, 1, 1, 0)])
@pytest.mark.parametrize("x_fmt,w_fmt", [((8, False), (8, True)), ((6, True), (4, True))])
def test_small_kernel_convolutions(x_fmt, w_fmt, geom):
    Bn, H, W, Cin, Cout, k, stride, pad = geom
    rng = np.random.default_rng(Cin + k)
    qx, qw = random_codes(rng, (Bn, H, W, Cin), x_fmt), random_codes(rng, (Cout, k, k, Cin), w_fmt)
    bias = rng.normal(0, 1, Cout).astype(np.float32)
    want, den = R.conv2d(qx, x_fmt, 0.3, qw, w_fmt, 0.02, stride, pad, bias, True)
    y_fmt, y_scale = (8, False), np.float32(np.abs(want).max() / R.vmax(8, False))
    args = (Bn, H, W, Cin, Cout, k, k, stride, pad, pack_rows_dev(qx.reshape(-1, Cin), x_fmt[0]), x_fmt, scalar(0.3),
            pack_rows_dev(qw.reshape(-1, Cin), w_fmt[0]), w_fmt, scalar(0.02))
    y, codes = B.dybit_conv2d_wb(*args, y_fmt, scalar(y_scale), dev(bias), None, True)
    assert B.dybit_last_gemm_kernel() == "f16_small"
    _, only = B.dybit_conv2d_wb(*args, y_fmt, scalar(y_scale), dev(bias), None, True, fp32=False)
    torch.cuda.synchronize()
    assert_within(y.cpu().numpy(), want, den)
    assert np.array_equal(codes.cpu().numpy().ravel(), R.quantize(y.cpu().numpy(), y_scale, *y_fmt).ravel())
    assert torch.equal(only, codes)


@pytest.mark.parametrize("fmts,shape,small", [(((8, False), (8, True)), (1024, 1024, 4096), True), (((8, False), (8, True)), (1024, 1088, 64), False),
                                              (((8, False), (8, True)), (1024, 1024, (1 << 14) + 4), False), (((8, False), (8, True)), (512, 1024, (1 << 14) + 4), True),
                                              (((4, False), (4, True)), (832, 512, 256), True), (((4, False), (4, True)), (832, 576, 256), False),
                                              (((4, False), (4, True)), (1216, 1216, 132), True), (((4, False), (4, True)), (1216, 1216, (1 << 14) + 4), False),
                                              (((8, False), (4, True)), (1024, 512, (1 << 19) + 64), True), (((8, False), (4, True)), (1024, 576, (1 << 19) + 64), False)])
def test_line_of_the_small_kernel(fmts, shape, small):
    """By tiles of 64 x 64, at half the line for a long K; code 1 everywhere: every sum is K."""
    M, N, K = shape
    (a_fmt, w_fmt), one = fmts, scalar(1.0)
    byte = lambda f: {8: 64 if f[1] else 128, 4: 0x44 if f[1] else 0x88}[f[0]]      # noqa: E731  codes of value 1
    a = torch.full((M * K * a_fmt[0] // 8,), byte(a_fmt), dtype=torch.uint8, device="cuda")
    w = torch.full((N * K * w_fmt[0] // 8,), byte(w_fmt), dtype=torch.uint8, device="cuda")
    c = B.dybit_gemm(M, N, K, a, a_fmt, one, w, w_fmt, one)
    assert ("small" in B.dybit_last_gemm_kernel()) == small
    assert bool((c == float(K)).all())
