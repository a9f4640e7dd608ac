"""The operand values that the benchmark feeds the loop of 6-bit matrix instructions: exactly the planes of the formats' values (no GPU)."""
import numpy as np
import pytest

import bench
from oracle import dybit_ref as R

SCALES = {(8, True): (4.0, 0.25), (6, False): (2.0, 0.5), (6, True): (1.0, 1.0)}


@pytest.mark.parametrize("fmt", [(8, True), (6, True), (6, False), (4, True), (4, False), (2, True), (2, False)])
def test_planes_make_up_every_value(fmt):
    values = np.asarray(R.codebook(*fmt), dtype=np.float64)
    mags = bench.e3m2_magnitudes()
    planes = bench.split_planes(values, fmt)
    total = sum(s * np.where(p & 32, -1, 1) * mags[p & 31] for p, s in zip(planes, SCALES.get(fmt, (1.0,)), strict=True))
    assert np.array_equal(total, values)


def test_ties_and_ends():
    code, value = bench.e3m2(np.array([0.0, 1 / 32, 3 / 32, 28.0, 100.0, -1.125, 1.375]))
    assert value.tolist() == [0.0, 0.0, 0.125, 28.0, 28.0, -1.0, 1.5] and code.tolist() == [0, 0, 2, 31, 31, 32 + 12, 14]


def test_lanes():
    codes = np.arange(64, dtype=np.uint8)
    lanes = bench.e3m2_lanes(codes)
    assert lanes.shape == (2, 32) and not lanes[:, 24:].any()
    bits = int.from_bytes(lanes[1].tobytes(), "little")
    assert [bits >> 6 * i & 63 for i in range(32)] == list(range(32, 64))
