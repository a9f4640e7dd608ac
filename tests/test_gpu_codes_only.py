"""Write-back calls that want codes only (no fp32 output) run on an epilogue of their own, over the transposed product:
its codes and its running maximum are those of the call that writes fp32 results as well, bit for bit (the fp32 results
and their codes are checked against the oracle in test_gpu_writeback.py)."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import dev, scalar, pack_rows_dev
from test_gpu_gemm import force_kernel, random_codes  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

OUT_FMTS = [(4, False), (4, True), (6, False), (6, True), (8, False), (8, True)]
KERNELS = ["ws", "mid1", "mid2", "mid64", "large", "mid1-f16"]


def both(args, tail, **kw):
    """(codes, maximum) of the call with both outputs and of the codes-only call; their fp32 results."""
    mx = torch.zeros(2, dtype=torch.float32, device="cuda")
    call = B.dybit_gemm_wb_rc if "r_codes" in kw else B.dybit_gemm_wb
    c, codes = call(*args, **kw, **tail, absmax=mx[0:1])
    guard = torch.full((codes.numel() + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    none, only = call(*args, **kw, **tail, absmax=mx[1:2], fp32=False, codes_out=guard[:codes.numel()])
    torch.cuda.synchronize()
    assert none is None and bool((guard[codes.numel():] == 0xA5).all())        # nothing past the last row
    assert torch.equal(only.reshape(-1), codes.reshape(-1))
    assert mx[0].item() == mx[1].item()
    return c


@pytest.mark.parametrize("force_kernel", KERNELS, indirect=True)
@pytest.mark.parametrize("c_fmt", OUT_FMTS)
@pytest.mark.parametrize("N", [64, 96, 208])                                   # one pair of column blocks; half a pair; a last group of 16 columns
@pytest.mark.parametrize("r_fmt", [None, (4, False), (6, True), (8, True), (8, False)])
def test_codes_only_equals_both_outputs(force_kernel, c_fmt, N, r_fmt):
    rng = np.random.default_rng(101 + N + c_fmt[0])
    a_fmt, w_fmt, M, K = (4, False), (4, True), 290, 128                        # 290: a last strip of two rows
    qa, qw = random_codes(rng, (M, K), a_fmt), random_codes(rng, (N, K), w_fmt)
    bias = rng.normal(0, 3, N).astype(np.float32)
    want, _ = R.gemm(qa, a_fmt, 0.37, qw, w_fmt, 0.011, bias, True)
    c_scale = np.float32(0.6 * np.abs(want).max() / R.vmax(*c_fmt))             # the largest results saturate
    args = (M, N, K, pack_rows_dev(qa, 4), a_fmt, scalar(0.37), pack_rows_dev(qw, 4), w_fmt, scalar(0.011), c_fmt, scalar(c_scale))
    kw = {}
    if r_fmt is not None:
        kw = {"r_codes": pack_rows_dev(random_codes(rng, (M, N), r_fmt), r_fmt[0]), "r_fmt": r_fmt, "r_scale": scalar(0.03)}
    for relu in (True, False):
        both(args, {"bias": dev(bias), "relu": relu}, **kw)
    both(args, {}, **kw)


@pytest.mark.parametrize("force_kernel", ["ws", "mid1", "mid64"], indirect=True)
@pytest.mark.parametrize("c_fmt", [(4, True), (6, True), (8, True)])
def test_codes_only_on_decision_points(force_kernel, c_fmt):
    """Every 4-bit unsigned times every 4-bit signed code, single products: hundreds of exact results on decision points."""
    a_fmt, w_fmt, K = (4, False), (4, True), 64
    qa, qw = np.zeros((256, K), dtype=np.uint8), np.zeros((64, K), dtype=np.uint8)
    qa[:, 5], qw[:, 5] = np.arange(256) % 16, np.arange(64) % 16
    ties = 0
    for c_scale in (0.5, 0.125, 0.0625):
        args = (256, 64, K, pack_rows_dev(qa, 4), a_fmt, scalar(1.0), pack_rows_dev(qw, 4), w_fmt, scalar(1.0), c_fmt, scalar(c_scale))
        c = both(args, {}).cpu().numpy()
        ties += np.isin(np.abs(c), R.midpoints(R.magnitude_bits(*c_fmt)) * c_scale).sum()
    assert ties > 100                                                           # the case is really there


@pytest.mark.parametrize("sa,sw,sc", [(2.0 ** 60, 2.0 ** 45, 2.0 ** 95), (2.0 ** -60, 2.0 ** -55, 2.0 ** -98), (1.0, 1.0, float("nan"))])
@pytest.mark.parametrize("force_kernel", ["ws", "mid1"], indirect=True)
def test_codes_only_extreme_scales(force_kernel, sa, sw, sc):
    """Scales whose product times the accumulators' power of two leaves the float range, and an unusable output scale."""
    rng = np.random.default_rng(5)
    a_fmt, w_fmt = (8, False), (8, True)
    qa, qw = random_codes(rng, (40, 64), a_fmt), random_codes(rng, (64, 64), w_fmt)
    codes = []
    for fp32 in (True, False):
        out = torch.full((40, 64), 7, dtype=torch.uint8, device="cuda")
        B.dybit_gemm_wb(40, 64, 64, pack_rows_dev(qa, 8), a_fmt, scalar(sa), pack_rows_dev(qw, 8), w_fmt, scalar(sw), (8, True), scalar(sc),
                        fp32=fp32, codes_out=out)
        torch.cuda.synchronize()
        assert B.dybit_get_last_async_error() == (B.OK if sc == sc else B.ERR_BAD_SCALE)
        codes.append(out)
    assert torch.equal(codes[0], codes[1])
    assert (sc == sc) or bool((codes[1] == 7).all())


@pytest.mark.parametrize("force_kernel", ["ws"], indirect=True)
@pytest.mark.parametrize("K", [192, 576, 704, 1216])                            # four, two and one workgroup's weights in a compute unit's LDS
@pytest.mark.parametrize("M", [31, 513, 1030])
def test_codes_only_by_lds_share(force_kernel, K, M):
    rng = np.random.default_rng(K)
    a_fmt, w_fmt, N = (8, False), (4, True), 64
    qa, qw = random_codes(rng, (M, K), a_fmt), random_codes(rng, (N, K), w_fmt)
    want, _ = R.gemm(qa, a_fmt, 0.37, qw, w_fmt, 0.011, None, True)
    args = (M, N, K, pack_rows_dev(qa, 8), a_fmt, scalar(0.37), pack_rows_dev(qw, 4), w_fmt, scalar(0.011), (6, False),
            scalar(np.abs(want).max() / R.vmax(6, False)))
    both(args, {"relu": True})
