"""Byte quantisation at lengths and alignments where four values a thread do
not fit, for one map and for a pair."""
import numpy as np
import pytest
import torch

import oracle
from paper_1703_02563_amd import learned as Lm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 2, 3, 4, 5, 1023, 1024, 1025, 4099, 1 << 20])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_equals_the_oracle(count, shift):
    rng = np.random.default_rng(count)
    a, b = (rng.normal(0, 3, count + shift).astype(np.float32) for _ in range(2))
    b[-1] = 40.0  # the pair's range comes from its second map, at the very end
    ta, tb = (torch.from_numpy(x).cuda()[shift:] for x in (a, b))
    a, b = a[shift:].copy(), b[shift:].copy()
    assert np.array_equal(Lm.quantize_u8(ta).cpu().numpy(), oracle.quantize_u8(a))
    for got, want in zip(Lm.quantize_pair_u8(ta, tb), oracle.quantize_pair_u8(a, b)):
        assert np.array_equal(got.cpu().numpy(), want)
