"""Scale images of two images in one launch: every scale against the oracle's
blur, at the edges of the 64 x 64 tiles and on frames smaller than a window."""
import numpy as np
import pytest
import torch

import oracle
from paper_1703_02563_amd import learned as Lm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,levels", [(1, 1, 1), (5, 3, 7), (64, 64, 7), (65, 127, 5), (63, 129, 3), (130, 200, 7)])
def test_every_scale_equals_the_oracle(H, W, levels):
    rng = np.random.default_rng(W + H)
    a, b = (rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))
    out = Lm.scale_images(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), levels).cpu().numpy()
    assert out.shape == (2 * levels, H, W)
    for k, img in enumerate((a, b)):
        for lv in range(levels):
            assert np.array_equal(out[k * levels + lv], oracle.blur(img, 1 << lv)), (k, lv)


def test_refused():
    a = torch.zeros((8, 9), dtype=torch.uint8, device="cuda")
    for args in ((a, a, 0), (a, a, 8), (a, a[:7].contiguous(), 3), (a, a[:, :8], 3), (a, a.float(), 3), (a, a.cpu(), 3)):
        with pytest.raises((RuntimeError, ValueError)):
            Lm.scale_images(*args)
