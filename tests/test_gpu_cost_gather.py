"""Gathered backward of the float patch cost at the sizes where its bins,
ranges and borders can go wrong: bit-exact against the fixed-point definition
(every term rounded to 2^-32 units, an exact integer sum, one rounding to
float32) evaluated in NumPy, whichever of the two forms the call takes."""
import numpy as np
import pytest
import torch

from paper_1703_02563_amd.learned import acc_scratch, cost_f32_grad

pytestmark = pytest.mark.gpu


def fixed_point_grad(f1, f2, ent, g, n, r):
    H, W, _ = f1.shape
    a1, a2 = (np.zeros((H * W, 16), np.int64) for _ in range(2))
    keep = g != 0
    ent, g2 = ent[keep].astype(np.int64), 2.0 * g[keep].astype(np.float64)
    x, y, fx, fy = ent.T
    for v in range(-r, r + 1):
        for u in range(-r, r + 1):
            p = np.clip(y + n * v, 0, H - 1) * W + np.clip(x + n * u, 0, W - 1)
            q = np.clip(y + fy + n * v, 0, H - 1) * W + np.clip(x + fx + n * u, 0, W - 1)
            d = g2[:, None] * (f1.reshape(-1, 16)[p].astype(np.float64) - f2.reshape(-1, 16)[q].astype(np.float64))
            t = np.rint(d * 2.0 ** 32).astype(np.int64)
            np.add.at(a1, p, t)
            np.add.at(a2, q, -t)
    return [(a.astype(np.float64) * 2.0 ** -32).astype(np.float32).reshape(H, W, 16) for a in (a1, a2)]


@pytest.mark.parametrize("W,H,n,r,count,place,scale", [
    (64, 48, 1, 3, 700, "inside", 1.0), (67, 41, 2, 3, 500, "inside", 1.0), (131, 70, 4, 4, 900, "inside", 1.0),
    (50, 40, 8, 3, 100, "inside", 1.0),                 # atomic form: n > 4
    (33, 29, 1, 0, 400, "inside", 1.0), (33, 29, 4, 0, 400, "inside", 1.0),
    (90, 80, 1, 7, 200, "inside", 1.0), (97, 83, 4, 7, 200, "inside", 1.0),
    (1, 200, 1, 3, 60, "inside", 1.0), (200, 1, 2, 2, 60, "inside", 1.0), (2, 3, 1, 3, 5, "inside", 1.0),
    (1, 1, 1, 0, 4, "inside", 1.0),
    (40, 30, 2, 3, 300, "outside", 1.0),                # centres and targets far outside the image
    (40, 30, 1, 3, 3000, "one", 1.0),                   # more than 2047 terms on a pixel
    (40, 30, 1, 2, 40, "inside", 3e5),                  # terms past 2^19: checked additions
    (16, 16, 1, 1, 5000, "inside", 1.0),                # too many entries for the bins: atomic form
])
def test_gradients_are_the_fixed_point_sums(W, H, n, r, count, place, scale):
    rng = np.random.default_rng(W * 1000 + H + n + r)
    f1, f2 = (rng.normal(size=(H, W, 16)).astype(np.float32) * np.float32(scale) for _ in range(2))
    x, y = rng.integers(0, W, count), rng.integers(0, H, count)
    fx, fy = rng.integers(-9, 10, count), rng.integers(-9, 10, count)
    if place == "outside":
        x, y = rng.integers(-60, W + 60, count), rng.integers(-60, H + 60, count)
        fx, fy = rng.integers(-90, 91, count), rng.integers(-90, 91, count)
    if place == "one":
        x[:], y[:] = W // 2, H // 2
    ent = np.stack([x, y, fx, fy], 1).astype(np.int32)
    g = rng.normal(size=count).astype(np.float32)
    g[::7] = 0.0
    want = fixed_point_grad(f1, f2, ent, g, n, r)
    acc = acc_scratch(W, H, "cuda")
    acc.fill_(-1)
    got = cost_f32_grad(*(torch.from_numpy(t).cuda() for t in (f1, f2, ent, g)), n, r, acc=acc)
    assert int(acc[-1]) == 0
    for a, b in zip(got, want):
        assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32))
