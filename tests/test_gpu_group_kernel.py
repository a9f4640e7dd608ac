"""Grouped convolutions that run as one launch (weight-stationary kernel, a group per workgroup), against the oracle: pieces of 8,
16 and 32 codes, groups of fewer and more than 32 and 64 output channels, filters whose K is no multiple of 64, ragged M."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import dev, scalar, pack_rows_dev, assert_within
from test_gpu_gemm import random_codes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("x_fmt,w_fmt", [((8, True), (4, True)), ((4, False), (6, True)), ((6, True), (8, True)), ((2, False), (2, True)), ((8, False), (8, True))])
@pytest.mark.parametrize("geom", [(2, 13, 11, 8, 8, 4, 3, 1, 1), (1, 20, 17, 16, 16, 2, 3, 2, 1), (3, 9, 9, 32, 32, 8, 3, 1, 1), (2, 8, 8, 32, 48, 2, 1, 1, 0),
                                  (1, 19, 23, 64, 72, 2, 3, 1, 1), (1, 9, 9, 16, 8, 3, 5, 1, 2), (1, 6, 50, 96, 64, 2, 1, 2, 0)])
@pytest.mark.parametrize("per_channel", [False, True])
def test_one_launch(x_fmt, w_fmt, geom, per_channel):
    Bn, H, W, cg, cog, groups, k, stride, pad = geom
    if (cg * w_fmt[0]) % 8:
        pytest.skip("filters start on a byte")
    rng = np.random.default_rng(cg + groups)
    Cin, Cout = cg * groups, cog * groups
    qx, qw = random_codes(rng, (Bn, H, W, Cin), x_fmt), random_codes(rng, (Cout, k, k, cg), w_fmt)
    bias = rng.normal(0, 1, Cout).astype(np.float32)
    sw = (rng.uniform(0.5, 2.0, Cout) * 0.02).astype(np.float32) if per_channel else np.full(1, 0.02, np.float32)
    parts = [R.conv2d(qx[..., i * cg:(i + 1) * cg], x_fmt, 0.3, qw[i * cog:(i + 1) * cog], w_fmt,
                      sw[i * cog:(i + 1) * cog] if per_channel else 0.02, stride, pad, bias[i * cog:(i + 1) * cog], True) for i in range(groups)]
    want, den = (np.concatenate([p[j] for p in parts], axis=3) for j in (0, 1))
    mx = torch.zeros(1, dtype=torch.float32, device="cuda")
    y = B.dybit_group_conv2d(Bn, H, W, Cin, Cout, k, k, stride, pad, groups, pack_rows_dev(qx.reshape(-1, Cin), x_fmt[0]), x_fmt, scalar(0.3),
                             pack_rows_dev(qw.reshape(Cout, -1), w_fmt[0]), w_fmt, dev(sw), dev(bias), None, True, mx, per_channel=per_channel)
    ran = B.dybit_last_gemm_kernel()
    torch.cuda.synchronize()
    assert (ran == "f16_group") == (cg * x_fmt[0] % 32 == 0)                    # else a group's channels are not whole words: a launch per group
    got = y.cpu().numpy()
    assert_within(got, want, den)
    assert mx.item() == np.abs(got).max()


def _sparse(n_bytes, at):
    """A tensor of zero bytes but for {position: value}."""
    q = torch.zeros(n_bytes, dtype=torch.uint8, device="cuda")
    for i, v in at.items():
        q[i] = v
    return q


def test_sizes_past_32_bits():
    """Sizes whose products leave 32 bits: every group's codes still meet its own filters.  Codes of value 1 in the last channels."""
    one = scalar(1.0)
    # filters of 2^30 codes (8 x 8 taps of 2^24 channels): no kernel's LDS holds them, a launch per group
    cg, fmt = 1 << 24, (2, True)
    x = _sparse(64 * 2 * cg // 4, {2 * cg // 4 - 1: 0x40, 64 * 2 * cg // 4 - 1: 0x55})     # pixel 0: the last channel; pixel 63: the last four
    w = _sparse(2 * 64 * cg // 4, {64 * cg // 4 + cg // 4 - 1: 0x40, 2 * 64 * cg // 4 - 1: 0x55})
    y = B.dybit_group_conv2d(1, 8, 8, 2 * cg, 2, 8, 8, 1, 0, 2, x, fmt, one, w, fmt, one)
    assert B.dybit_last_gemm_kernel() != "f16_group" and y.flatten().tolist() == [0.0, 5.0]
    del x, w
    # a pixel of 2^29 channels: the groups' channels start beyond 2^32 bits
    groups, cg, fmt = 1 << 19, 1024, (8, False)
    v = R.codebook(*fmt)
    x = _sparse(groups * cg, {groups * cg - 1: 200, groups // 2 * cg: 100})
    w = torch.zeros(groups, cg, dtype=torch.uint8, device="cuda")
    w[:, 0], w[:, -1] = 3, 5
    y = B.dybit_group_conv2d(1, 1, 1, groups * cg, groups, 1, 1, 1, 0, groups, x, fmt, one, w.reshape(-1), (8, True), one).flatten()
    s = R.codebook(8, True)
    assert B.dybit_last_gemm_kernel() == "f16_group"
    assert y[-1].item() == np.float32(v[200] * s[5]) and y[groups // 2].item() == np.float32(v[100] * s[3]) and int((y != 0).sum()) == 2
    del x, w
    # 2^20 groups: one launch for them would be 2^32 threads
    groups, cg, fmt = 1 << 20, 8, (4, False)
    x = _sparse(groups * cg // 2, {groups * cg // 2 - 1: 0x70, 0: 0x07})
    w = torch.full((groups * cg // 2,), 0x11, dtype=torch.uint8, device="cuda")
    y = B.dybit_group_conv2d(1, 1, 1, groups * cg, groups, 1, 1, 1, 0, groups, x, fmt, one, w, (4, True), one).flatten()
    want = np.float32(R.codebook(*fmt)[7] * R.codebook(4, True)[1])
    assert y[0].item() == want and y[-1].item() == want and int((y != 0).sum()) == 2
