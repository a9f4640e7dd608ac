"""3 x 3 windows at stride 2 on codes, the kernel whose threads walk strips of output rows: edges of images and strips."""
import numpy as np
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from test_gpu_pool import FMTS, packed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 3, 3), (2, 4, 7), (1, 15, 16), (3, 18, 5), (2, 33, 40)])
def test_strips(fmt, pad, shape):
    """One output row and column, strips with one to four rows left, odd and even images, several images in a workgroup."""
    Bn, H, W = shape
    if H + 2 * pad < 3 or W + 2 * pad < 3:
        pytest.skip("window larger than the padded image")
    rng = np.random.default_rng(H * 50 + W + fmt[0])
    C = 32 // fmt[0]
    q = rng.integers(0, 1 << fmt[0], (Bn, H, W, C)).astype(np.uint8)
    if fmt[1]:
        q[:, ::3] = 1 << (fmt[0] - 1)                          # negative zeros: written as the all-zero code
        q[0] = rng.integers(1 << (fmt[0] - 1), 1 << fmt[0], (H, W, C))   # an image of negative values only
    got = B.dybit_maxpool2d_codes(Bn, H, W, C, 3, 2, pad, packed(q, fmt[0]), fmt)
    torch.cuda.synchronize()
    want = R.maxpool2d_codes(q, *fmt, 3, 2, pad)
    assert np.array_equal(got.cpu().numpy().reshape(-1), R.pack_rows(want.reshape(-1, C), fmt[0]).reshape(-1))
