"""Blurred images of ff_descriptors at patch scales that are no power of two (the
sub-scales 3n/2) and at the ends of the range, against the oracle: random frames
and frames of 255, whose window sums are the largest."""
import numpy as np
import pytest
import torch

import oracle
import paper_1703_02563_amd as ff

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 5, 6, 12, 24, 33, 48, 63, 64])
@pytest.mark.parametrize("H,W", [(1, 1), (5, 70), (66, 63), (130, 131)])
def test_blurred_equals_the_oracle(H, W, n):
    rng = np.random.default_rng(H * W + n)
    frames = [rng.integers(0, 256, (H, W), dtype=np.uint8), np.full((H, W), 255, np.uint8)]
    frames.append(np.where(rng.random((H, W)) < 0.5, 255, 254).astype(np.uint8))
    for img in frames:
        assert np.array_equal(ff.descriptors(torch.from_numpy(img).cuda(), n)[0].cpu().numpy(), oracle.blur(img, n))
