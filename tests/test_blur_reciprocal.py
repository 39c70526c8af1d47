"""The blur's rounded mean by a 32-bit reciprocal: exact for every sum of every
window (half-widths 1 .. 32)."""
import numpy as np
import pytest


@pytest.mark.parametrize("h", range(1, 33))
def test_reciprocal_is_exact(h):
    area = (2 * h + 1) ** 2
    x = np.arange(255 * area + area // 2 + 1, dtype=np.uint64)
    q = (x * np.uint64(0xFFFFFFFF // area + 1)) >> np.uint64(32)
    assert np.array_equal(q, x // np.uint64(area))
