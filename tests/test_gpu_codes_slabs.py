"""Codes-only products with more rows than the persistent grid of the weight-stationary kernels takes at once: a slab's first codes are
requested while the slab in front of it is encoded.  Bit for bit the codes of the call that writes fp32 results as well, which requests nothing ahead."""
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import scalar
from test_gpu_codes_only import both
from test_gpu_gemm import force_kernel  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SLABS = 256 * 16 * 32                                                          # rows that the waves of a full device hold at once (64 columns)


@pytest.mark.parametrize("force_kernel", ["ws"], indirect=True)
@pytest.mark.parametrize("a_fmt,w_fmt", [((4, False), (8, True)), ((8, False), (6, True)), ((6, True), (4, True)), ((4, True), (4, True))])
@pytest.mark.parametrize("K", [64, 128, 192, 320])                             # one step, the two requested ahead, odd and more
@pytest.mark.parametrize("M,N,r_fmt", [(SLABS + 45, 64, None), (SLABS // 2 + 3, 208, (8, False)), (2 * SLABS + 7, 96, None)])
def test_every_slab(force_kernel, a_fmt, w_fmt, K, M, N, r_fmt):
    gen = torch.Generator(device="cuda").manual_seed(K + M + N)
    draw = lambda rows, cols, fmt: torch.randint(0, 256, (rows * cols * fmt[0] // 8,), dtype=torch.uint8, device="cuda", generator=gen)
    a, w = draw(M, K, a_fmt), draw(N, K, w_fmt)
    sa, sw = scalar(0.37), scalar(0.011)
    top = B.dybit_gemm(M, N, K, a, a_fmt, sa, w, w_fmt, sw).abs().max()
    kw = {"r_codes": draw(M, N, r_fmt), "r_fmt": r_fmt, "r_scale": (top / 64).reshape(1)} if r_fmt else {}
    c_fmt = (4, True) if K == 128 else (6, False)
    both((M, N, K, a, a_fmt, sa, w, w_fmt, sw, c_fmt, (0.6 * top / R.vmax(*c_fmt)).reshape(1)), {"relu": True}, **kw)
