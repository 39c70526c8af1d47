"""Gathered backward of the float patch cost where many entries meet on few
pixels: inside the image (pixels on both sides of the 256 terms that one quad
sums), on a corner, along an edge.  The gradients are the fixed-point sums
bit for bit, and the call takes no longer than the atomic form (which maps
that are not 16-byte aligned take)."""
import numpy as np
import pytest
import torch

from paper_1703_02563_amd.learned import acc_scratch, cost_f32_grad
from test_gpu_cost_gather import fixed_point_grad

pytestmark = pytest.mark.gpu


def crowd(place, W, H, count, rng):
    x, y = rng.integers(0, W, count), rng.integers(0, H, count)
    fx, fy = rng.integers(-9, 10, count), rng.integers(-9, 10, count)
    if place == "pixel":
        x[:], y[:] = W // 2, H // 2
    elif place == "corner":
        x[:], y[:], fx[:], fy[:] = W - 1, 0, 0, 0
    elif place == "edge":
        y[:], fy[:] = H - 1, 0
    elif place == "column":
        x[:], fx[:] = 0, 0
    elif place == "patch":
        x, y = W // 2 + rng.integers(0, 8, count), H // 2 + rng.integers(0, 8, count)
    return np.stack([x, y, fx, fy], 1).astype(np.int32), rng.normal(size=count).astype(np.float32)


@pytest.mark.parametrize("W,H,n,r,count,place,scale", [
    (64, 48, 1, 3, 256, "pixel", 1.0), (64, 48, 1, 3, 257, "pixel", 1.0), (64, 48, 2, 1, 4000, "pixel", 1.0),
    (67, 53, 4, 7, 700, "pixel", 1.0), (64, 48, 1, 3, 900, "pixel", 3e5),
    (160, 140, 1, 0, 140000, "pixel", 1.0),  # more than 2047 terms for each of a workgroup's 64 quads
    (64, 48, 1, 3, 900, "corner", 1.0), (67, 53, 4, 2, 900, "corner", 1.0), (40, 30, 2, 0, 900, "corner", 1.0),
    (64, 48, 1, 3, 1500, "edge", 1.0), (67, 53, 4, 3, 1500, "edge", 1.0), (53, 67, 2, 2, 1500, "column", 1.0),
    (96, 64, 1, 3, 4000, "patch", 1.0), (1, 160, 1, 1, 600, "edge", 1.0), (160, 1, 2, 1, 600, "column", 1.0),
    (2, 80, 1, 1, 500, "patch", 1.0), (80, 2, 1, 1, 500, "spread", 1.0),
])
def test_gradients_are_the_fixed_point_sums(W, H, n, r, count, place, scale):
    rng = np.random.default_rng(W * 1000 + H + n + r + count)
    f1, f2 = (rng.normal(size=(H, W, 16)).astype(np.float32) * np.float32(scale) for _ in range(2))
    ent, g = crowd(place, W, H, count, rng)
    want = fixed_point_grad(f1, f2, ent, g, n, r)
    acc = acc_scratch(W, H, "cuda")
    acc.fill_(-1)
    got = cost_f32_grad(*(torch.from_numpy(t).cuda() for t in (f1, f2, ent, g)), n, r, acc=acc)
    assert int(acc[-1]) == 0
    for a, b in zip(got, want):
        assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("place", ["pixel", "corner", "edge", "patch"])
def test_a_term_out_of_range_is_seen(place):
    W, H, rng = 64, 48, np.random.default_rng(3)
    f1, f2 = (torch.from_numpy(rng.normal(size=(H, W, 16)).astype(np.float32)).cuda() for _ in range(2))
    ent, g = crowd(place, W, H, 900, rng)
    g[450] = 1e30
    acc = acc_scratch(W, H, "cuda")
    got = cost_f32_grad(f1, f2, torch.from_numpy(ent).cuda(), torch.from_numpy(g).cuda(), 1, 3, acc=acc)
    assert int(acc[-1]) != 0 and all(bool(torch.isnan(t).all()) for t in got)


@pytest.mark.parametrize("W,H,count,place", [
    (160, 120, 16384, "pixel"), (160, 120, 16384, "corner"), (160, 120, 16384, "edge"), (160, 120, 65536, "patch"),
    (64, 48, 2048, "corner"), (64, 48, 8192, "spread"),
])
def test_not_slower_than_the_atomic_form(W, H, count, place):
    rng = np.random.default_rng(5)
    ent, g = (torch.from_numpy(t).cuda() for t in crowd(place, W, H, count, rng))
    acc = acc_scratch(W, H, "cuda")

    def best_us(off):
        f = [torch.randn(H * W * 16 + off, device="cuda")[off:].view(H, W, 16) for _ in range(2)]
        out = tuple(torch.empty(H, W, 16, device="cuda") for _ in range(2))
        times = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            cost_f32_grad(*f, ent, g, 1, 3, out=out, acc=acc)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 1e3)
        return min(times[1:])

    gather, atomic = best_us(0), best_us(1)
    assert gather <= 1.2 * atomic, (gather, atomic)
