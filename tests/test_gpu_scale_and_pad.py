"""Scales of tensors around the sizes where dybit_absmax_scale changes its launches (one workgroup; a workspace of partial
maxima; past the last-level cache), and the encoder that pads three channels to four, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import dev, scalar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 3, 4, 4095, 32768 * 4 + 1, 65535, 65536, 65537, 65540, 1 << 20, (1 << 22) + 3])
def test_scale_with_and_without_workspace(n):
    rng = np.random.default_rng(n)
    x = rng.normal(0, 1, n).astype(np.float32)
    xd = dev(x)
    own = torch.cuda.current_stream()
    for at in {0, n // 2, n - 1} if n else {None}:                          # the maximum first, in the middle, last; then a NaN there
        if at is not None:
            xd = dev(x)
            xd[at] = -7.5
        for special in (None, float("nan")) if at is not None else (None,):
            if special is not None:
                xd[at] = special
            want = R.absmax_scale(np.nan_to_num(xd.cpu().numpy(), nan=0.0), 4, True)
            out = torch.full((1,), float("nan"), device="cuda")             # what was there before does not matter
            a = B.dybit_absmax_scale(xd, 4, True, out=out)
            b = B.dybit_absmax_scale(xd, 4, True, stream=own)
            torch.cuda.synchronize()
            assert a.item() == want and b.item() == want


def test_scale_of_a_tensor_beyond_the_cache():
    n = (1 << 26) + 5
    x = torch.full((n,), 0.25, device="cuda")
    for at in (0, n // 3, n - 1):
        x[at] = -3.0
        assert B.dybit_absmax_scale(x, 8, True).item() == 3.0 / 64
        x[at] = 0.25
    assert B.dybit_absmax_scale(torch.zeros(70000, device="cuda"), 8, True).item() == 1.0


@pytest.mark.parametrize("fmt", [(2, True), (4, True), (6, False), (6, True), (8, True)])
@pytest.mark.parametrize("rows", [1, 3, 4, 5, 1023, 4096, 5001])
def test_pad_three_channels(fmt, rows):
    rng = np.random.default_rng(rows)
    x = rng.normal(0, 1, (rows, 3)).astype(np.float32)
    s = np.float32(np.abs(x).max() / R.vmax(*fmt) * 0.9)
    x.ravel()[:: max(1, x.size // 7)] = s * R.midpoints(R.magnitude_bits(*fmt))[0]   # decision points among them
    got = B.dybit_quantize_pad(dev(x), 4, scalar(s), *fmt)
    torch.cuda.synchronize()
    padded = np.concatenate([x, np.zeros((rows, 1), np.float32)], axis=1)
    assert np.array_equal(got.cpu().numpy().ravel(), R.pack(R.quantize(padded, s, *fmt).ravel(), fmt[0]))
