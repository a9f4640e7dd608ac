"""Products on split operands (6-bit floats): every format pair the kernel takes, at the edges of its tiles, units and row
ends, against the oracle.  Parity is exact equality: the planes hold every value, their products and the sums of these cases
fit fp32 (K times the largest product below 2^24 steps), so nothing rounds.  Results with a bias: the product tolerance."""
import numpy as np
import pytest

from oracle import dybit_ref as R
from gpu_util import assert_within, dev, oracle_codes, pack_rows_dev, scalar
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


@pytest.mark.parametrize("larger", ["+++", "++-", "++", "+-"])
@pytest.mark.parametrize("a_fmt,w_fmt", PAIRS)
def test_several_largest_products_beside_a_smaller_one(tile, a_fmt, w_fmt, larger):
    """Every code of A times every code of W in one group of four k with two or three products of the largest values, of either sign: the
    instruction adds a group at the place of its largest product, and nothing of the smaller one may go."""
    top_a, top_w = (1 << (a_fmt[0] - a_fmt[1])) - 1, (1 << (w_fmt[0] - 1)) - 1
    M, N, K = 4 << a_fmt[0], 1 << w_fmt[0], 64
    qa, qw = np.zeros((M, K), np.uint8), np.zeros((N, K), np.uint8)
    for p in range(4):                                           # a group for each position of the smaller product; a row of A uses one of them
        group = [16 * p + 4 + j for j in range(4)]
        small = group.pop(p)
        qa[p::4, small], qw[:, small] = np.arange(1 << a_fmt[0]), np.arange(N)
        for k, sign in zip(group, larger):
            qa[p::4, k], qw[:, k] = top_a, top_w | (1 << (w_fmt[0] - 1) if sign == "-" else 0)
    got = product(M, N, K, qa, a_fmt, qw, w_fmt).cpu().numpy()
    assert B.dybit_last_gemm_kernel() == tile
    want, _ = R.gemm(qa, a_fmt, 1.0, qw, w_fmt, 1.0)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("a_fmt,w_fmt", [((8, True), (4, True)), ((6, False), (4, True)), ((4, True), (8, True)), ((4, False), (4, True)), ((2, False), (2, True))])
def test_long_sums_of_positive_products(tile, a_fmt, w_fmt):
    """Nothing cancels and the sum outgrows its terms by 2^15: what the fp32 sums round, which is within the product's tolerance."""
    M, N, K = 130, 70, 1 << 15
    rng = np.random.default_rng(K + a_fmt[0])
    qa, qw = rng.integers(1, 1 << (a_fmt[0] - a_fmt[1]), (M, K)).astype(np.uint8), rng.integers(1, 1 << (w_fmt[0] - 1), (N, K)).astype(np.uint8)
    got = product(M, N, K, qa, a_fmt, qw, w_fmt).cpu().numpy()
    assert B.dybit_last_gemm_kernel() == tile
    want, den = R.gemm(qa, a_fmt, 1.0, qw, w_fmt, 1.0)
    assert_within(got, want, den)


def work_call(M, N, K, a, a_fmt, w, w_fmt, out, work, work_bytes, scale):
    assert B.lib().dybit_gemm_work(M, N, K, a.data_ptr(), B.fmt(*a_fmt), scale.data_ptr(), w.data_ptr(), B.fmt(*w_fmt), scale.data_ptr(), None, 0,
                                   out.data_ptr(), out.shape[1], work, work_bytes, B._stream(None)) == B.OK
    return B.dybit_last_gemm_kernel()


def test_entry_point_with_a_workspace():
    """dybit_gemm_work itself: what it does with less memory than it asks for, none, or some that does not begin on 16 bytes, with rows of results too
    far apart, and that it keeps to the bytes it asks for."""
    import torch
    M, N, K, a_fmt, w_fmt = 3000, 2000, 1532, (8, True), (4, True)
    need = int(B.lib().dybit_gemm_workspace_bytes(M, N, K, B.fmt(*a_fmt), B.fmt(*w_fmt)))
    rng = np.random.default_rng(8)
    a, w = pack_rows_dev(rng.integers(0, 256, (M, K)).astype(np.uint8), 8), pack_rows_dev(rng.integers(0, 16, (N, K)).astype(np.uint8), 4)
    one, out = scalar(1.0), torch.empty(M, N, device="cuda")
    args = (M, N, K, a, a_fmt, w, w_fmt)
    guard = 4096
    memory = torch.full((need + 2 * guard,), 0xa5, dtype=torch.uint8, device="cuda")
    at = memory.data_ptr() + guard
    assert at % 16 == 0
    assert work_call(*args, out, at, need, one) == "f6_128"
    assert (memory[:guard] == 0xa5).all() and (memory[guard + need:] == 0xa5).all() and not (memory[guard:guard + need] == 0xa5).all()
    memory.fill_(0xff)                                           # no contents matter
    again = torch.empty_like(out)
    assert work_call(*args, again, at, need + guard, one) == "f6_128" and torch.equal(out, again)
    memory.fill_(0xa5)
    for pointer, size in ((at, need - 1), (at, 0), (None, need), (at + 8, need), (at + 1, need)):
        other = torch.empty_like(out)
        assert work_call(*args, other, pointer, size, one).startswith("f16_128")
        assert torch.equal(other, out)                           # integers below 2^24 steps of 2^-8: exact on either kernel
    assert (memory == 0xa5).all()


def test_rows_of_results_too_far_apart():
    import torch
    M, N, K, a_fmt, w_fmt, ldc = 130, 200, 2048, (8, True), (4, True), 1 << 23
    rng = np.random.default_rng(9)
    qa, qw = rng.integers(0, 256, (M, K)).astype(np.uint8), rng.integers(0, 16, (N, K)).astype(np.uint8)
    a, w, one = pack_rows_dev(qa, 8), pack_rows_dev(qw, 4), scalar(1.0)
    out = torch.empty(M, ldc, device="cuda")                     # 4.4 GB
    memory = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    B.dybit_set_option("gemm_kernel", "six")
    try:
        need = int(B.lib().dybit_gemm_workspace_bytes(M, N, K, B.fmt(*a_fmt), B.fmt(*w_fmt)))
        assert 0 < need <= memory.numel()
        assert not work_call(M, N, K, a, a_fmt, w, w_fmt, out, memory.data_ptr(), need, one).startswith("f6")
    finally:
        B.dybit_set_option("gemm_kernel", "auto")
    want, den = R.gemm(qa, a_fmt, 1.0, qw, w_fmt, 1.0)
    assert_within(out[:, :N].cpu().numpy(), want, den)


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
    taken = []
    try:
        with pytest.raises(torch.cuda.OutOfMemoryError):         # what other tests have left in the allocator's segments as well
            while True:
                taken.append(torch.empty(need, dtype=torch.uint8, device="cuda"))
        assert B.dybit_gemm(*args, out=out) is out
        assert B.dybit_last_gemm_kernel() == "f16_256"
    finally:
        taken.clear()
        torch.cuda.set_per_process_memory_fraction(1.0)
    # the same products in another order of summation: 2^-24 of sum |a b| for each of the K / 16 steps that add into a result, at most
    bound = (K / 16 + 1) * 2.0 ** -24 * 0.125 * K * 64 * 4
    assert (out - want).abs().max().item() <= bound
    assert B.dybit_gemm(*args).equal(want) and B.dybit_last_gemm_kernel() == "f6_256"


@pytest.mark.parametrize("a_bits,before", [(8, "f16_256"), (4, "f8_256")])
def test_8192_cubed_on_either_kernel(a_bits, before):
    """The benchmark's 8192^3 products: as a call takes them, and on the kernel that callers without a workspace get; the oracle evaluates a
    sample of rows and columns exactly."""
    import torch
    from paper_2302_12510_amd import synth
    size, a_fmt, w_fmt = 8192, (a_bits, True), (4, True)
    cfg = synth.config5a(size=size)
    (sa, qa), (sw, qw) = oracle_codes(cfg["A"], a_fmt), oracle_codes(cfg["W"], w_fmt)
    a, w = pack_rows_dev(qa, a_bits), pack_rows_dev(qw, 4)
    rng = np.random.default_rng(a_bits)
    rows, cols = (np.unique(np.concatenate([[0, 127, 128, 255, 256, size - 1], rng.integers(0, size, n)])) for n in (60, 508))
    want, den = R.gemm(qa[rows], a_fmt, sa, qw[cols], w_fmt, sw)
    for option, kernel in (("auto", "f6_256"), ("large", before)):
        B.dybit_set_option("gemm_kernel", option)
        try:
            c = B.dybit_gemm(size, size, size, a, a_fmt, scalar(sa), w, w_fmt, scalar(sw))
        finally:
            B.dybit_set_option("gemm_kernel", "auto")
        assert B.dybit_last_gemm_kernel() == kernel
        assert_within(c[torch.from_numpy(rows).cuda()][:, torch.from_numpy(cols).cuda()].cpu().numpy(), want, den)


@pytest.mark.parametrize("a_fmt,w_fmt", [((8, True), (4, True)), ((4, True), (8, True)), ((2, False), (8, True))])
@pytest.mark.parametrize("K", [32768, 32772])
def test_tiles_of_128_keep_two_sums(a_fmt, w_fmt, K):
    """Sums of positive products that outgrow 2^24 steps of theirs, but no half of them does: the halves (128 k in turn) are exact, as the two
    k-groups of the kernel such products ran on are, and the result is their sum rounded once."""
    M, N = 70, 130
    a_bits, w_bits = a_fmt[0] - a_fmt[1], w_fmt[0] - 1
    step = 2.0 ** (1 - a_bits) * 2.0 ** (1 - w_bits)
    rng = np.random.default_rng(K + a_fmt[0])
    qa, qw = (rng.integers(0, 1 << b, s) for b, s in ((a_bits, (M, K)), (w_bits, (N, K))))
    value_a, value_w = (R.codebook(*f)[:1 << b].astype(np.float64) for f, b in ((a_fmt, a_bits), (w_fmt, w_bits)))
    mean = K * value_a.mean() * value_w.mean() / step
    if mean < 1.4 * 2 ** 24:                                     # more of the largest codes, until the mean is 1.4 * 2^24 steps
        top = value_a[-1] * value_w[-1] * K / step
        share = (1.4 * 2 ** 24 - mean) / (top - mean)
        k = rng.random(K) < share
        qa[:, k], qw[:, k] = (1 << a_bits) - 1, (1 << w_bits) - 1
    qa, qw = qa.astype(np.uint8), qw.astype(np.uint8)
    turn = np.arange(K) // 128 % 2
    halves = [np.asarray(R.gemm(qa[:, turn == t], a_fmt, 1.0, qw[:, turn == t], w_fmt, 1.0)[0], dtype=np.float64) for t in (0, 1)]
    assert max(h.max() for h in halves) < 2 ** 24 * step < (halves[0] + halves[1]).min()
    B.dybit_set_option("gemm_kernel", "six")
    B.dybit_set_option("mid_tile", "128")
    try:
        got = product(M, N, K, qa, a_fmt, qw, w_fmt).cpu().numpy()
    finally:
        B.dybit_set_option("gemm_kernel", "auto")
        B.dybit_set_option("mid_tile", "auto")
    assert B.dybit_last_gemm_kernel() == "f6_128"
    assert np.array_equal(got, (halves[0] + halves[1]).astype(np.float32))
