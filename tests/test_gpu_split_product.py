"""Products on split operands (6-bit floats): every format pair the kernel takes, at the edges of its tiles, units and row
ends, against the oracle.  Parity is exact equality: the planes hold every value, their products and the sums of these cases
fit fp32 (K times the largest product below 2^24 steps), so nothing rounds.  Results with a bias: the product tolerance."""
import numpy as np
import pytest

from oracle import dybit_ref as R
from gpu_util import assert_within, dev, pack_rows_dev, scalar
from paper_2302_12510_amd import binding as B

pytestmark = pytest.mark.gpu

ONE = [(4, True), (2, True)]
TWO = [(8, True), (6, True)]
PAIRS = ([(a, w) for a in TWO + [(6, False), (4, True), (4, False), (2, True), (2, False)] for w in ONE]
         + [(a, w) for a in [(4, True), (2, True), (2, False)] for w in TWO])


@pytest.fixture(params=["128", "256"])
def tile(request):
    B.dybit_set_option("gemm_kernel", "six")
    B.dybit_set_option("mid_tile", "128" if request.param == "128" else "auto")
    yield "f6_" + request.param
    B.dybit_set_option("gemm_kernel", "auto")
    B.dybit_set_option("mid_tile", "auto")


def product(M, N, K, qa, a_fmt, qw, w_fmt, bias=None, relu=False, **kw):
    return B.dybit_gemm(M, N, K, pack_rows_dev(qa, a_fmt[0]), a_fmt, scalar(1.0), pack_rows_dev(qw, w_fmt[0]), w_fmt, scalar(1.0),
                        None if bias is None else dev(bias), relu, **kw)


@pytest.mark.parametrize("shape", [(1, 1, 4), (33, 65, 68), (128, 128, 128), (130, 257, 192), (257, 129, 388), (300, 520, 640)])
@pytest.mark.parametrize("a_fmt,w_fmt", PAIRS)
def test_exact(tile, a_fmt, w_fmt, shape):
    M, N, K = shape
    rng = np.random.default_rng(M + N + K + a_fmt[0] + w_fmt[0])
    qa, qw = (rng.integers(0, 1 << f[0], s).astype(np.uint8) for f, s in ((a_fmt, (M, K)), (w_fmt, (N, K))))
    got = product(M, N, K, qa, a_fmt, qw, w_fmt).cpu().numpy()
    assert B.dybit_last_gemm_kernel() == tile
    want, _ = R.gemm(qa, a_fmt, 1.0, qw, w_fmt, 1.0)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("a_fmt,w_fmt", PAIRS)
def test_largest_and_smallest_products_meet(tile, a_fmt, w_fmt):
    """Every code of A against every code of W beside the product of the largest two, at each position of a group of four k."""
    top_a, top_w = (1 << (a_fmt[0] - a_fmt[1])) - 1, (1 << (w_fmt[0] - 1)) - 1
    M, N, K = 4 << a_fmt[0], 1 << w_fmt[0], 64
    qa, qw = np.zeros((M, K), np.uint8), np.zeros((N, K), np.uint8)
    qa[:, 8], qw[:, 8] = top_a, top_w
    for m in range(M):
        qa[m, 9 + m % 4] = m // 4
    for j in range(4):
        qw[:, 9 + j] = np.arange(N)
    got = product(M, N, K, qa, a_fmt, qw, w_fmt).cpu().numpy()
    assert B.dybit_last_gemm_kernel() == tile
    want, _ = R.gemm(qa, a_fmt, 1.0, qw, w_fmt, 1.0)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("ldc_extra", [0, 3])
@pytest.mark.parametrize("relu", [False, True])
def test_bias_relu_and_row_pitch(tile, relu, ldc_extra):
    M, N, K, a_fmt, w_fmt = 261, 139, 1532, (8, True), (4, True)
    rng = np.random.default_rng(5)
    qa, qw = rng.integers(0, 256, (M, K)).astype(np.uint8), rng.integers(0, 16, (N, K)).astype(np.uint8)
    bias = rng.normal(0, 50, N).astype(np.float32)
    out = dev(np.full((M, N + ldc_extra), 7.0, np.float32))
    got = product(M, N, K, qa, a_fmt, qw, w_fmt, bias, relu, out=out, ldc=N + ldc_extra).cpu().numpy()
    assert B.dybit_last_gemm_kernel() == tile
    want, den = R.gemm(qa, a_fmt, 1.0, qw, w_fmt, 1.0, bias, relu)
    assert_within(got[:, :N], want, den)
    assert (got[:, N:] == 7.0).all()


def test_one_stream_after_another_and_capture():
    """The workspace comes from the current stream's allocator; a captured call replays with eager work in between."""
    import torch
    M, N, K, a_fmt, w_fmt = 3000, 2000, 1532, (8, True), (4, True)
    assert B.lib().dybit_gemm_workspace_bytes(M, N, K, B.fmt(*a_fmt), B.fmt(*w_fmt)) > 0
    rng = np.random.default_rng(6)
    args = (M, N, K, pack_rows_dev(rng.integers(0, 256, (M, K)).astype(np.uint8), 8), a_fmt, scalar(0.5),
            pack_rows_dev(rng.integers(0, 16, (N, K)).astype(np.uint8), 4), w_fmt, scalar(0.25))
    want = B.dybit_gemm(*args)
    assert B.dybit_last_gemm_kernel().startswith("f6")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    out = torch.empty_like(want)
    with torch.cuda.stream(side):
        B.dybit_gemm(*args)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            B.dybit_gemm(*args, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        assert torch.equal(B.dybit_gemm(*args), want)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    # a stream that is not the current one has no workspace to use: the product runs as without one
    B.dybit_gemm(*args, out=out, stream=side)
    assert not B.dybit_last_gemm_kernel().startswith("f6")
    side.synchronize()
    assert torch.allclose(out, want, rtol=1e-5, atol=1e-2)


def test_no_memory_for_a_workspace():
    """A product whose workspace the allocator refuses runs as without one."""
    import torch
    M, N, K, a_fmt, w_fmt = 4096, 4096, 4096, (8, True), (4, True)
    need = B.lib().dybit_gemm_workspace_bytes(M, N, K, B.fmt(*a_fmt), B.fmt(*w_fmt))
    gen = torch.Generator(device="cuda").manual_seed(7)
    args = (M, N, K, torch.randint(0, 256, (M * K,), dtype=torch.uint8, device="cuda", generator=gen), a_fmt, scalar(0.5),
            torch.randint(0, 256, (N * K // 2,), dtype=torch.uint8, device="cuda", generator=gen), w_fmt, scalar(0.25))
    want, out = B.dybit_gemm(*args), torch.zeros(M, N, device="cuda")
    assert B.dybit_last_gemm_kernel() == "f6_256"
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + need // 4) / total)
    try:
        with pytest.raises(torch.cuda.OutOfMemoryError):
            torch.empty(need, dtype=torch.uint8, device="cuda")
        assert B.dybit_gemm(*args, out=out) is out
        assert B.dybit_last_gemm_kernel() == "f16_256"
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    # the same products in another order of summation: 2^-24 of sum |a b| for each of the K / 16 steps that add into a result, at most
    bound = (K / 16 + 1) * 2.0 ** -24 * 0.125 * K * 64 * 4
    assert (out - want).abs().max().item() <= bound
    assert B.dybit_gemm(*args).equal(want) and B.dybit_last_gemm_kernel() == "f6_256"
