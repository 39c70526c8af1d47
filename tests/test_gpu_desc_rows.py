"""Descriptor and weight-class maps at row widths and bases of every alignment,
rows shorter than a phase, sub-scales, and a frame whose rows only just fit in LDS."""
import numpy as np
import pytest
import torch

import paper_1703_02563_amd as ff
from paper_1703_02563_amd.ffi import check, lib
from paper_1703_02563_amd.flowfields import _ptr, _stream

pytestmark = pytest.mark.gpu


def columns(n, Wp):
    """col(c) of every padded column (phase order; image order where n is no power of two)."""
    c = np.arange(Wp)
    if n & (n - 1):
        return c
    return (c % n) * (Wp // n) + np.minimum(c % n, Wp % n) + c // n


@pytest.mark.parametrize("W,H,n,shift", [
    (1, 1, 1, 0), (1, 3, 16, 0), (5, 4, 8, 1), (63, 5, 64, 0), (64, 9, 1, 0), (65, 9, 2, 3), (66, 7, 4, 2),
    (67, 7, 8, 1), (130, 6, 16, 0), (257, 5, 32, 2), (1030, 3, 1, 1), (101, 6, 3, 1), (90, 5, 24, 0),
    (12900, 2, 1, 0), (12800, 2, 64, 3), (32766, 1, 2, 1),
])
def test_maps_equal_the_definition(W, H, n, shift):
    rng = np.random.default_rng(W * 64 + n)
    img = torch.from_numpy(rng.integers(0, 256, (H, W), dtype=np.uint8)).cuda()
    P = 4 * n
    hsum = torch.empty((H, W), dtype=torch.int16, device="cuda")
    blurred = torch.empty(H * W + 4, dtype=torch.uint8, device="cuda")[shift:shift + H * W].view(H, W)
    desc = torch.empty((H + 2 * P, W + 2 * P, 16), dtype=torch.uint8, device="cuda")
    plain = torch.empty((H, W, 16), dtype=torch.uint8, device="cuda")
    wf = torch.empty((H + 6 * n, W, 16), dtype=torch.uint8, device="cuda")
    check(lib().ff_descriptors(_ptr(img), W, H, n, _ptr(hsum), _ptr(blurred), _ptr(desc), _ptr(plain), _ptr(wf),
                               _stream()), "ff_descriptors")
    b = blurred.cpu().numpy()
    ys, xs = np.arange(H), np.arange(W)
    want = np.empty((H, W, 16), np.uint8)
    for gy in range(4):
        for gx in range(4):
            want[..., 4 * gy + gx] = b[np.clip(ys + n * (2 * gy - 3), 0, H - 1)[:, None],
                                       np.clip(xs + n * (2 * gx - 3), 0, W - 1)[None]]
    assert np.array_equal(plain.cpu().numpy(), want)
    yc, xc = np.clip(np.arange(H + 2 * P) - P, 0, H - 1), np.clip(np.arange(W + 2 * P) - P, 0, W - 1)
    padded = np.empty((H + 2 * P, W + 2 * P, 16), np.uint8)
    padded[:, columns(n, W + 2 * P)] = want[yc][:, xc]
    assert np.array_equal(desc.cpu().numpy(), padded)
    # weight-class rows: bytes -6 -5 5 6 | -4 -3 3 4 | -2 -1 1 2 | 0, samples n apart, clamped
    offs = (-6, -5, 5, 6, -4, -3, 3, 4, -2, -1, 1, 2, 0)
    w = wf.cpu().numpy()
    rows = b[np.clip(np.arange(H + 6 * n) - 3 * n, 0, H - 1)]
    for k, a in enumerate(offs):
        assert np.array_equal(w[..., k], rows[:, np.clip(xs + n * a, 0, W - 1)]), a
    assert not w[..., 13:].any()
