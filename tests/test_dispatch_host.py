"""Which kernel a call would start, seen without a GPU: the dispatcher runs on the host and notes the kernel before the launch, which then
fails for want of a device.  Pointers are made up, so nothing here runs where there is a device."""
import ctypes as C

import pytest
import torch

from paper_2302_12510_amd import binding as B

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="made-up pointers must never reach a device")
P, NULL = C.c_void_p(0x10000), C.c_void_p(0)


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
    assert st == B.ERR_HIP
    return B.dybit_last_gemm_kernel()


def test_stride_beyond_the_image(option):
    """Images of one row of one output, 2^20 pixels from one to the next: 127 of them never fit the LDS, however far 2^30 columns of stride reach
    (their product with the bytes of a pixel leaves 64 bits)."""
    assert not conv_kernel(127, 1, 1 << 20, 64, 8, 1, 2, 1 << 30, 0, 2, 4).endswith("_patch")
