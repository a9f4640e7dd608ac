"""The native argument marshalling of the binding (no GPU needed: every call here is refused before it launches anything)."""
import re
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
