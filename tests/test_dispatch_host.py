"""Which kernel a call would start, seen without a GPU: the dispatcher runs on the host and notes the kernel before the launch, which then
fails for want of a device.  Pointers are made up, so nothing here runs where there is a device."""
import ctypes as C
import os
import subprocess
import sys

import pytest
import torch

from paper_2302_12510_amd import binding as B

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="made-up pointers must never reach a device")
P, NULL = C.c_void_p(0x10000), C.c_void_p(0)
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(params=["auto", "patch"])
def option(request):
    B.dybit_set_option("gemm_kernel", request.param)
    yield request.param
    B.dybit_set_option("gemm_kernel", "auto")


def conv_kernel(Bn, H, W, cin, cout, kh, kw, stride, pad, a_bits, w_bits, out="fp32"):
    """out: fp32, codes (4-bit), both (fp32 and 4-bit codes)."""
    assert B.lib().dybit_set_async_error_word(P) == B.OK
    st = B.lib().dybit_conv2d_wb(Bn, H, W, cin, cout, kh, kw, stride, pad, P, B.fmt(a_bits, False), P, P, B.fmt(w_bits, True), P, NULL, NULL, 1,
                                 NULL if out == "codes" else P, NULL, B.fmt(4, False), P, NULL if out == "fp32" else P, None)
    assert B.lib().dybit_set_async_error_word(NULL) == B.OK
    assert st in (B.OK, B.ERR_HIP)
    return B.dybit_last_gemm_kernel()


def test_stride_beyond_the_image(option):
    """Images of one row of one output, 2^20 pixels from one to the next: 127 of them never fit the LDS, however far 2^30 columns of stride reach
    (their product with the bytes of a pixel leaves 64 bits)."""
    assert not conv_kernel(127, 1, 1 << 20, 64, 8, 1, 2, 1 << 30, 0, 2, 4).endswith("_patch")


#  B   H   W  Cin Cout kh kw s  p  A  W -> whether the many-channel kernel is taken
@pytest.mark.parametrize("geom,takes", [
    ((1, 400, 400, 64, 64, 3, 3, 1, 1, 8, 4), False), ((1, 400, 400, 64, 64, 3, 3, 1, 1, 4, 4), False), ((4, 112, 112, 64, 64, 3, 3, 1, 1, 4, 4), True),    # wide images
    ((69, 75, 32, 384, 128, 1, 3, 1, 0, 8, 8), False), ((69, 75, 32, 384, 128, 1, 5, 1, 0, 8, 8), True),                                                    # filters of one row
    ((64, 56, 56, 64, 128, 3, 3, 2, 1, 4, 4), False), ((64, 56, 56, 128, 256, 3, 3, 2, 1, 4, 4), True), ((32, 60, 90, 128, 256, 3, 3, 3, 0, 4, 4), False),   # strides
    ((2, 40, 40, 64, 160, 1, 2, 1, 0, 8, 8), False), ((2, 40, 40, 64, 256, 2, 2, 1, 0, 6, 4), False), ((2, 40, 40, 128, 256, 2, 2, 1, 0, 6, 4), True),       # K
    ((62, 8, 7, 64, 200, 1, 2, 1, 0, 8, 4), False), ((16, 64, 64, 64, 1024, 3, 1, 1, 0, 8, 4), False),
    ((16, 39, 17, 256, 160, 3, 3, 2, 1, 4, 2), False), ((16, 39, 17, 256, 160, 3, 3, 1, 1, 4, 2), True), ((16, 39, 17, 64, 160, 5, 5, 2, 2, 4, 2), True), ((64, 14, 14, 256, 512, 3, 3, 2, 1, 4, 4), True)])                                                   # 64 x 64 tiles
@pytest.mark.parametrize("out", ["fp32", "codes"])
def test_taps_that_share_pixels(geom, takes, out):
    """The kernel pays where a pixel that it decodes once serves several taps: not for wide images, long strides, two or three taps or a short K."""
    assert conv_kernel(*geom, out=out).endswith("_patch") == takes


@pytest.mark.parametrize("geom,takes", [
    ((64, 7, 7, 512, 512, 3, 3, 1, 1, 8, 8), True), ((64, 7, 7, 512, 512, 3, 3, 1, 1, 4, 4), True),                                                  # tiles of 128; of 64, 392 of them
    ((20, 16, 16, 64, 128, 3, 3, 1, 1, 2, 2), False), ((36, 16, 16, 128, 128, 3, 3, 1, 1, 4, 4), True),                                              # tiles of 64: 160 and 288
    ((9, 33, 33, 256, 64, 5, 5, 1, 2, 4, 4), True), ((9, 33, 33, 256, 64, 3, 3, 1, 1, 4, 4), False), ((40, 14, 14, 128, 96, 3, 3, 1, 1, 8, 6), True),   # K
    ((40, 14, 14, 128, 96, 3, 3, 1, 1, 8, 4), False), ((40, 14, 14, 128, 96, 3, 3, 1, 1, 8, 8), False), ((40, 14, 14, 192, 96, 3, 3, 1, 1, 8, 8), True),   # small outputs
    ((13, 56, 56, 64, 64, 3, 3, 1, 1, 8, 4), False), ((64, 56, 56, 64, 64, 3, 3, 1, 1, 2, 2), False), ((13, 56, 56, 128, 64, 3, 3, 1, 1, 4, 4), True),     # stationary weights
    ((13, 56, 56, 64, 96, 3, 3, 1, 1, 8, 4), True), ((32, 40, 40, 64, 160, 7, 1, 1, 0, 8, 8), False)])                                                # columns; K
def test_both_outputs(geom, takes):
    """Calls that write fp32 results and codes have the long epilogue: the kernel is taken less often for them."""
    assert conv_kernel(*geom, out="both").endswith("_patch") == takes


@pytest.mark.parametrize("geom,outs", [
    ((53, 90, 90, 64, 64, 3, 3, 1, 0, 8, 4), ""), ((14, 91, 91, 128, 64, 3, 3, 1, 0, 8, 4), ""), ((64, 56, 56, 64, 64, 3, 3, 1, 1, 8, 4), "fp32 codes"),       # few taps a pixel; 4.8
    ((7, 127, 127, 128, 160, 3, 3, 1, 0, 2, 4), ""), ((2, 127, 127, 128, 160, 3, 3, 1, 0, 2, 4), "fp32 codes both"),                                     # 856 tiles; 490
    ((53, 90, 90, 64, 160, 3, 3, 1, 0, 2, 4), "fp32 codes both"), ((53, 90, 90, 128, 160, 3, 3, 1, 0, 2, 4), ""),                                        # strips of 39 KiB; of 70
    ((64, 56, 56, 128, 256, 3, 3, 2, 1, 4, 4), "fp32 codes"), ((73, 20, 128, 192, 64, 3, 3, 1, 0, 4, 4), ""), ((30, 90, 90, 128, 64, 3, 3, 1, 0, 4, 4), "fp32 codes both"),   # 4-bit pair
    ((30, 90, 90, 128, 32, 3, 3, 1, 0, 2, 4), "fp32 codes both"), ((30, 90, 90, 128, 40, 3, 3, 1, 0, 2, 4), "")])                                        # columns
def test_many_tiles(geom, outs):
    """Many tiles of long strips whose pixels serve few taps are left to the kernels with more workgroups a compute unit."""
    assert [out for out in ("fp32", "codes", "both") if conv_kernel(*geom, out=out).endswith("_patch")] == outs.split()


@pytest.mark.parametrize("geom,outs", [
    ((16, 22, 22, 128, 512, 3, 3, 2, 1, 6, 4), "codes"), ((38, 26, 26, 128, 128, 3, 3, 2, 1, 8, 2), "codes"), ((29, 35, 34, 64, 64, 3, 3, 2, 1, 8, 6), "fp32 codes"),   # stride 2
    ((1, 56, 56, 256, 256, 3, 3, 1, 1, 8, 4), "fp32 codes"), ((2, 7, 129, 192, 320, 3, 3, 1, 1, 8, 4), "codes"), ((2, 40, 40, 64, 160, 3, 3, 1, 0, 6, 6), "fp32 codes both"),   # share
    ((6, 26, 72, 320, 40, 3, 2, 1, 0, 2, 4), ""), ((2, 60, 60, 64, 64, 3, 3, 1, 1, 4, 4), "fp32 codes"), ((2, 70, 70, 64, 64, 3, 3, 1, 0, 4, 4), "codes"),          # tiles of 64: share 1.8; 4.6; 2.8
    ((55, 17, 17, 512, 64, 3, 2, 1, 0, 2, 4), "fp32 codes"), ((9, 33, 33, 256, 64, 5, 5, 1, 2, 4, 4), "fp32 codes both")])
def test_few_tiles(geom, outs):
    """Against the kernels for few tiles it needs more taps a pixel, and stride 1 where they decode with more waves."""
    assert [out for out in ("fp32", "codes", "both") if conv_kernel(*geom, out=out).endswith("_patch")] == outs.split()


@pytest.mark.parametrize("cin,a_bits,w_bits,takes", [(192, 6, 6, True), (192, 2, 8, True), (192, 8, 6, True), (192, 8, 8, False), (192, 4, 8, False), (256, 6, 6, False), (256, 8, 6, False)])
@pytest.mark.parametrize("out", ["fp32", "codes", "both"])
def test_what_the_large_tiles_decline(cin, a_bits, w_bits, takes, out):
    """6- and 8-bit weights are left to the 256 x 256 kernel, but it takes 6- and 2-bit operands only with whole groups of 128 channels."""
    assert conv_kernel(64, 28, 28, cin, 192, 3, 3, 1, 1, a_bits, w_bits, out).endswith("_patch") == takes


# Stands between the library and the runtime: prints what a call asks for and launches nothing.
SHIM = """
#include <cstdio>
struct Dim { unsigned x, y, z; };
extern "C" int hipFuncSetAttribute(const void *f, int what, int value) { std::printf("limit %p %d\\n", f, value); std::fflush(stdout); return 0; }
extern "C" int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *) { std::printf("launch %u %u %zu\\n", grid.x, block.x, lds); std::fflush(stdout); return 1; }
"""
PRELUDE = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)                     # found before the runtime's own
sys.path[:0] = [sys.argv[2], sys.argv[2] + "/tests"]
import test_dispatch_host as T
from paper_2302_12510_amd import binding as B
P, f8 = T.P, B.fmt(8, True)
"""


@pytest.fixture
def asked(tmp_path):
    """Runs Python lines on a library that launches nothing; the words of every line printed."""
    (tmp_path / "shim.cpp").write_text(SHIM)
    shim = str(tmp_path / "shim.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", str(tmp_path / "shim.cpp"), "-o", shim], check=True)

    def run(lines):
        p = subprocess.run([sys.executable, "-c", PRELUDE + lines, shim, ROOT], capture_output=True, text=True)
        assert p.returncode == 0, p.stderr
        return [line.split() for line in p.stdout.splitlines()]
    return run


CALLS = """
for out in ("fp32", "codes"):
    for option, calls in (("patch", [(4, 14, 14, 64, 64, 3, 3, 1, 1, 8, 8), (4, 28, 28, 128, 64, 3, 3, 1, 1, 8, 8)]),
                          ("few", [(64, 112, 112, 4, 64, 7, 7, 2, 3, 8, 8), (64, 224, 224, 4, 64, 7, 7, 2, 3, 8, 8), (64, 64, 64, 8, 64, 3, 3, 1, 1, 8, 8)]),
                          ("ws", [(64, 28, 28, 64, 64, 3, 3, 1, 1, 4, 4), (64, 28, 28, 128, 64, 3, 3, 1, 1, 4, 4), (64, 28, 28, 64, 64, 3, 3, 1, 1, 8, 8), (64, 28, 28, 64, 64, 1, 1, 1, 0, 8, 8)])):
        B.dybit_set_option("gemm_kernel", option)
        for c in calls:
            assert option in T.conv_kernel(*c, out=out)
    B.dybit_set_option("gemm_kernel", "auto")
for cin, cout, k in ((256, 256, 3), (512, 256, 3), (512, 256, 1)):
    B.lib().dybit_group_conv2d(4, 14, 14, cin, cout, k, k, 1, k // 2, 8, P, f8, P, P, f8, P, 0, None, None, 0, P, None, None)
for k, stride in ((5, 1), (5, 2), (7, 2)):
    B.lib().dybit_dwconv2d(4, 28, 28, 32, k, k, stride, k // 2, P, f8, P, P, f8, P, None, 0, P, None, None)
"""


def test_lds_limits_are_constants(asked):
    """The LDS limit of a kernel belongs to the whole process: every call sets the same one, or two threads with different sizes could
    set it against each other between one's setting and its launch."""
    limits, launches = {}, 0
    for word, *rest in asked(CALLS):
        if word == "limit":
            limits.setdefault(rest[0], []).append(int(rest[1]))
        launches += word == "launch"
    assert launches == 24 and sum(map(len, limits.values())) == launches and len(limits) < launches
    assert all(len(set(v)) == 1 and 64 * 1024 <= v[0] <= 160 * 1024 for v in limits.values()), limits


@pytest.mark.parametrize("geom", [(8, 256, 708, 4, 64, 7, 7, 2, 3, 8, 8), (16, 250, 250, 16, 64, 2, 2, 1, 0, 8, 8), (4, 256, 736, 4, 64, 8, 8, 2, 3, 8, 8), (64, 224, 224, 4, 64, 7, 7, 2, 3, 8, 8)])
def test_few_channel_walkers_fit_the_device(asked, geom):
    """Its workgroups walk over the units of work, as many of them as 256 compute units hold at once: each has 256 bytes of LDS of its own beside
    what the launch asks for (codes out)."""
    lines = asked(f'B.dybit_set_option("gemm_kernel", "few")\nassert T.conv_kernel(*{geom}, out="codes") == "f16_few"')
    (grid, threads, lds), = [map(int, rest) for word, *rest in lines if word == "launch"]
    per_cu = min(160 * 1024 // (lds + 256), 1024 // threads)
    assert grid <= 256 * per_cu
