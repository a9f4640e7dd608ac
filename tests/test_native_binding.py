"""The native argument marshalling of the binding, and ctypes in its place where it cannot be imported (no GPU needed, but for
the last test: every other call here is refused before it launches anything)."""
import re
import sys
from pathlib import Path

import numpy as np
import pytest
import torch

from paper_2302_12510_amd import binding as B

NATIVE = B._n()
CPU = torch.zeros(64)


def test_every_entry_checks_its_argument_count():
    header = (Path(__file__).parents[1] / "include" / "dybit.h").read_text()
    names = [n for n in dir(NATIVE) if n.startswith("dybit_")]
    assert len(names) == 27
    for n in names:
        assert re.search(rf"\b{n}\(", header)
        with pytest.raises(TypeError, match="arguments"):
            getattr(NATIVE, n)()


def test_what_the_binding_refuses():
    with pytest.raises(ValueError, match="expected a device tensor"):
        B.dybit_quantize(CPU, CPU[:1], 4, True, out=torch.zeros(32, dtype=torch.uint8))
    with pytest.raises(ValueError, match="expected a device tensor"):
        B.dybit_gemm(1, 1, 16, CPU, (4, True), CPU, CPU, (4, True), CPU)
    with pytest.raises(AssertionError):
        B.dybit_quantize(CPU.double(), CPU[:1], 4, True)
    with pytest.raises(AttributeError):
        NATIVE.dybit_quantize("x", 1, (4, True), None, None, None)
    for pair in ((4,), (4, True, 1), "ab", 4):
        with pytest.raises((TypeError, ValueError)):
            NATIVE.dybit_quantize(None, 1, pair, None, None, _Stream())
    with pytest.raises(AttributeError):
        NATIVE.dybit_quantize(None, 0, (4, True), None, None, 7)         # not a stream


class _Stream:
    cuda_stream = 0


@pytest.mark.parametrize("bits,signed,status", [(4, True, B.ERR_NULL), (5, True, B.ERR_UNSUPPORTED_BITS), (np.int64(4), np.bool_(True), B.ERR_NULL),
                                                (4.0, 1, B.ERR_NULL)])
def test_arguments_reach_the_library(bits, signed, status):
    assert NATIVE.dybit_quantize(None, 16, (bits, signed), None, None, _Stream()) == status
    assert NATIVE.dybit_quantize(None, np.int64(16), [bits, signed], None, None, _Stream()) == status


def test_allocations():
    t = NATIVE.empty(CPU, True, 3, 5)
    assert t.dtype == torch.float32 and t.shape == (3, 5) and t.device == CPU.device
    assert NATIVE.empty(CPU, False, 7).dtype == torch.uint8
    assert NATIVE.dybit_packed_bytes((6, True), 9) == 7


@pytest.fixture
def without_native(monkeypatch):
    monkeypatch.setattr(B, "_native_module", None)
    monkeypatch.setitem(sys.modules, B.__package__ + "._native", None)          # its import now fails
    monkeypatch.delattr(sys.modules[B.__package__], "_native", raising=False)


def test_without_the_native_module(without_native):
    with pytest.warns(RuntimeWarning, match="native argument marshalling"):
        n = B._n()
    assert n is not NATIVE and B._n() is n
    with pytest.raises(ValueError, match="expected a device tensor"):
        B.dybit_gemm(1, 1, 16, CPU, (4, True), CPU, CPU, (4, True), CPU)
    for pair, status in (((4, True), B.ERR_NULL), ((5, True), B.ERR_UNSUPPORTED_BITS), ([np.int64(4), np.bool_(True)], B.ERR_NULL)):
        assert n.dybit_quantize(None, np.int64(16), pair, None, None, _Stream()) == status
    assert n.empty(CPU, True, 3, 5).shape == (3, 5) and n.empty(CPU, False, 7).dtype == torch.uint8
    assert n.dybit_packed_bytes((6, True), 9) == 7


def test_arguments_are_converted_once():
    """Also by the product's wrapper, which looks at some of them itself."""
    seen = []

    class Index:
        def __init__(self, name, value):
            self.name, self.value = name, value

        def __index__(self):
            seen.append(self.name)
            return self.value

    class Bits(Index):
        def __int__(self):
            return self.__index__()

    with pytest.raises(ValueError, match="expected a device tensor"):
        NATIVE.dybit_gemm(Index("M", 64), Index("N", 64), Index("K", 256), None, (Bits("a", 4), True), None, None, (Bits("w", 4), True), None,
                          None, False, CPU, 64, None)
    assert seen == ["M", "N", "K", "a", "w"]


@pytest.mark.gpu
@pytest.mark.filterwarnings("ignore:the native argument marshalling")
def test_results_without_the_native_module(without_native):
    x = torch.randn(64, 256, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    def chain():
        s = B.dybit_absmax_scale(x.reshape(-1), 4, True)
        q = B.dybit_quantize(x.reshape(-1), s, 4, True)
        word = torch.zeros(1, device="cuda")
        return s, q, B.dybit_gemm_ex(64, 64, 256, q, (4, True), s, q, (4, True), s, absmax=word, relu=True), word
    by_ctypes = chain()
    B._native_module = NATIVE
    for a, b in zip(by_ctypes, chain()):
        assert torch.equal(a, b)
