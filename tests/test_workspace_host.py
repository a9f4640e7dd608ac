"""Which products ask for a workspace, and how much (host code: no GPU)."""
import pytest

from paper_2302_12510_amd import binding as B

UNIT = 3072                                                  # bytes of 32 rows x 128 k as 6-bit floats


def need(M, N, K, a, w):
    return int(B.lib().dybit_gemm_workspace_bytes(M, N, K, B.fmt(*a), B.fmt(*w)))


@pytest.mark.parametrize("a,w,planes", [((8, True), (4, True), (2, 1)), ((6, False), (2, True), (2, 1)), ((4, True), (8, True), (1, 2)),
                                        ((4, False), (4, True), (1, 1)), ((2, True), (6, True), (1, 2))])
def test_bytes(a, w, planes):
    M, N, K = 8000, 4001, 4100
    units = lambda rows: (rows + 31) // 32 * ((K + 127) // 128)  # noqa: E731
    assert need(M, N, K, a, w) == UNIT * (planes[0] * units(M) + planes[1] * units(N))


@pytest.mark.parametrize("a,w", [((8, False), (4, True)),        # three planes
                                 ((8, True), (8, True)), ((6, True), (6, True)),   # four pairs of planes
                                 ((4, False), (8, True)), ((4, False), (6, True)),   # products span more than the instruction keeps
                                 ((8, True), (4, False)), ((5, True), (4, True))])
def test_declined_formats(a, w):
    assert need(8192, 8192, 8192, a, w) == 0


def test_sizes():
    a, w = (8, True), (4, True)
    assert need(8192, 8192, 8192, a, w) and need(2999, 1999, 1532, a, w)
    assert not need(2999, 1999, 1000, a, w) and not need(512, 512, 8192, a, w) and not need(32768, 64, 4096, a, w)
    assert not need(0, 100, 100, a, w) and not need(1 << 20, 1 << 20, 8192, a, w)      # nothing to do; codes of 2 GiB and more
    assert need(4096, 4096, 4096, (4, True), w) and not need(2048, 2688, 960, (4, True), w) and need(2048, 2688, 964, (4, True), w)


def test_options_leave_it_out():
    a, w = (8, True), (4, True)
    for name, value in (("gemm_kernel", "large"), ("gemm_mfma", "f16"), ("mid_tile", "128"), ("mid_kgroups", "1"), ("gemm_ws", "off")):
        B.dybit_set_option(name, value)
        try:
            assert need(8192, 8192, 8192, a, w) == 0
        finally:
            B.dybit_set_option(name, "auto")
    assert need(8192, 8192, 8192, a, w)

