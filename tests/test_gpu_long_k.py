"""Products whose rows of codes are so long that 32-bit counts of codes or bits would overflow: every code of K counts (a row of zeros
with a few codes set at its start, in its middle and at its end; the sum is exact)."""
import pytest
import torch

from oracle import dybit_ref as R
from paper_2302_12510_amd import binding as B
from gpu_util import scalar

pytestmark = pytest.mark.gpu


def sparse_row(K, bits, at):
    """Packed zero codes, all-ones magnitudes of a signed format at the positions `at`."""
    q = torch.zeros(K * bits // 8, dtype=torch.uint8, device="cuda")
    for k in at:
        for b in range(bits - 1):
            q[(k * bits + b) // 8] |= 1 << ((k * bits + b) % 8)
    return q


@pytest.mark.parametrize("bits,K", [(6, 360_000_000), (6, 358_000_004), (2, 1 << 31), (8, (1 << 28) + 192)])
def test_single_row(bits, K):
    fmt, at = (bits, True), [3, K // 2, K - 70, K - 2]
    a, w, one = sparse_row(K, bits, at + [7]), sparse_row(K, bits, at + [9]), scalar(1.0)
    c = B.dybit_gemm(1, 1, K, a, fmt, one, w, fmt, one)
    ran = B.dybit_last_gemm_kernel()
    assert c.item() == len(at) * R.vmax(*fmt) ** 2
    assert ran not in ("f16_small", "f8_small")                                # whose counts are 32-bit
