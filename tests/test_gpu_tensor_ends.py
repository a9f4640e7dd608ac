"""Tensors of codes that end inside a 32-bit word (rows that start at any byte): their last one to three bytes count, the bytes
behind them do not, on every kernel that fetches such tensors by whole words, against the oracle; and one tensor of
2^31 - 2 bytes, the largest that those kernels take."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import dev, scalar, pack_rows_dev, assert_within
from test_gpu_gemm import random_codes
from test_gpu_small_ragged import kernel  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def ending(codes2d, bits, behind):
    """The packed rows at the start of a larger buffer of `behind` bytes."""
    packed = pack_rows_dev(codes2d, bits).reshape(-1)
    buf = torch.full((packed.numel() + 64,), behind, dtype=torch.uint8, device="cuda")
    buf[:packed.numel()] = packed
    return buf[:packed.numel()]


@pytest.mark.parametrize("a_fmt,w_fmt,K", [((8, True), (8, True), 197), ((8, False), (4, True), 198), ((6, True), (6, True), 196), ((4, False), (2, True), 204),
                                           ((2, True), (8, True), 68), ((4, False), (4, True), 1150)])
@pytest.mark.parametrize("M,N", [(31, 33), (33, 31), (129, 65)])
def test_products(kernel, a_fmt, w_fmt, K, M, N):
    rng = np.random.default_rng(M * 7 + K)
    qa, qw = random_codes(rng, (M, K), a_fmt), random_codes(rng, (N, K), w_fmt)
    qa[-1, -9:], qw[-1, -9:] = (1 << R.magnitude_bits(*a_fmt)) - 1, (1 << R.magnitude_bits(*w_fmt)) - 1    # the last codes weigh most
    want, den = R.gemm(qa, a_fmt, 0.37, qw, w_fmt, 0.011)
    got = []
    for behind in (0xFF, 0x5A):
        c = B.dybit_gemm(M, N, K, ending(qa, a_fmt[0], behind), a_fmt, scalar(0.37), ending(qw, w_fmt[0], behind), w_fmt, scalar(0.011))
        assert B.dybit_last_gemm_kernel() != "general"
        torch.cuda.synchronize()
        got.append(c.cpu().numpy())
    assert_within(got[0], want, den)
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("x_fmt,w_fmt", [((6, False), (6, True)), ((4, True), (4, True)), ((6, True), (2, True))])
def test_few_channel_convolution(x_fmt, w_fmt):
    Bn, H, W, Cin, Cout = 1, 97, 103, 4, 19                                     # 9991 pixels; 19 filters of 196 codes
    rng = np.random.default_rng(19)
    qx, qw = random_codes(rng, (Bn, H, W, Cin), x_fmt), random_codes(rng, (Cout, 7, 7, Cin), w_fmt)
    want, den = R.conv2d(qx, x_fmt, 0.3, qw, w_fmt, 0.02, 2, 3)
    got = []
    for behind in (0xFF, 0x5A):
        x, w = ending(qx.reshape(-1, Cin), x_fmt[0], behind), ending(qw.reshape(Cout, -1), w_fmt[0], behind)
        assert x.numel() % 4 and w.numel() % 4
        got.append(B.dybit_conv2d(Bn, H, W, Cin, Cout, 7, 7, 2, 3, x, x_fmt, scalar(0.3), w, w_fmt, scalar(0.02)).cpu().numpy())
        assert B.dybit_last_gemm_kernel() == "f16_few"
    assert_within(got[0], want, den)
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("w_fmt,k", [((6, True), 3), ((2, True), 1), ((2, True), 3)])
def test_grouped_convolution(w_fmt, k):
    x_fmt, cg, cog, groups = (8, False), 8, 3, 3
    rng = np.random.default_rng(k)
    qx, qw = random_codes(rng, (1, 9, 7, cg * groups), x_fmt), random_codes(rng, (cog * groups, k, k, cg), w_fmt)
    want, den = R.group_conv2d(qx, x_fmt, 0.3, qw, w_fmt, 0.02, 1, k // 2, groups)
    got = []
    for behind in (0xFF, 0x5A):
        w = ending(qw.reshape(cog * groups, -1), w_fmt[0], behind)
        assert w.numel() % 4
        got.append(B.dybit_group_conv2d(1, 9, 7, cg * groups, cog * groups, k, k, 1, k // 2, groups, pack_rows_dev(qx.reshape(-1, cg * groups), 8), x_fmt,
                                        scalar(0.3), w, w_fmt, scalar(0.02)).cpu().numpy())
        assert B.dybit_last_gemm_kernel() == "f16_group"
    assert_within(got[0], want, den)
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("large", ["activations", "weights"])
def test_largest_tensor(large):
    """3243933 rows of 662 bytes are 2^31 - 2: the last two bytes, whose word ends at 2^31, count."""
    rows, K, few, fmt = 3243933, 662, 8, (8, True)
    rng = np.random.default_rng(5)
    tail, small = random_codes(rng, (40, K), fmt), random_codes(rng, (few, K), fmt)
    tail[-1, :] = 0
    tail[-1, -2:] = (127, 126)                                                  # the last row is its last two codes
    small[:, -2:] = (101, 17)
    q = torch.zeros(rows * K, dtype=torch.uint8, device="cuda")
    q[-40 * K:] = dev(tail).reshape(-1)
    one = scalar(1.0)
    if large == "activations":
        c = B.dybit_gemm(rows, few, K, q, fmt, one, dev(small), fmt, one)[-40:]
        want, den = R.gemm(tail, fmt, 1.0, small, fmt, 1.0)
    else:
        c = B.dybit_gemm(few, rows, K, dev(small), fmt, one, q, fmt, one)[:, -40:]
        want, den = R.gemm(small, fmt, 1.0, tail, fmt, 1.0)
    assert B.dybit_last_gemm_kernel() == "f16_128_kg1"
    torch.cuda.synchronize()
    assert_within(c.cpu().numpy(), want, den)
