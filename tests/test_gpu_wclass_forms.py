"""The weight-class kernels beside the plain radius-3 one (subpixel flows,
sub-scale stages, patch radii 2 and 4) on every tile they come in, bit-exact
against the oracle on frames whose interior (cells and targets the patch
radius away from the border) is empty, one pixel wide, or larger than a tile;
and the tables chosen by grid size against the same call with an explicit
table."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_1703_02563_amd as ff

pytestmark = pytest.mark.gpu
NT = max(1, min(8, os.cpu_count() or 1))
KEYS = ("flow_fwd", "flow_bwd", "cost_fwd", "cost_bwd", "keep_fwd", "keep_bwd")
FORMS = {"subpixel": (dict(subpixel=3), dict(subpixel=3)),
         "subscales": (dict(subscales=True), dict(subscales=True)),
         "radius2": (dict(radius=2), dict(radius=2)), "radius4": (dict(radius=4), dict(radius=4))}


def frames(seed, H, W):
    rng = np.random.default_rng(seed)
    a = rng.integers(0, 256, (H, W))
    b = np.roll(a, (1, -2), (0, 1)) + rng.integers(-3, 4, (H, W))
    return a.astype(np.uint8), np.clip(b, 0, 255).astype(np.uint8)


def same(got, want, n_evals=None):
    for k in KEYS:
        g, w = got[k].cpu().numpy(), want[k]
        w = w.cpu().numpy() if isinstance(w, torch.Tensor) else w
        assert np.array_equal(g.view(w.dtype) if g.dtype != w.dtype else g, w), k
    want_n = want["n_evals"]
    want_n = want_n.cpu().tolist() if isinstance(want_n, torch.Tensor) else list(want_n)
    assert got["n_evals"].cpu().tolist() == want_n


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("W,H", [(67, 50), (25, 24), (13, 7)])
def test_every_tile_equals_the_oracle(form, W, H):
    kw, okw = FORMS[form]
    a, b = frames(W + H, H, W)
    L, T, r = 3, 4, okw.get("radius", 3)
    ref = oracle.flow_fields(a, b, L, T, r, nthreads=NT, **{k: v for k, v in okw.items() if k != "radius"})
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    for v in (31, 11, 30, 26, 27, 32, 14):  # one table index per tile
        tun = ff.default_tuning().replace(variant=[v] * 7, passes=[0] * 7)
        same(ff.flow_fields(da, db, ff.Params(levels=L, iters=T, tuning=tun, **kw)), ref)


@pytest.mark.parametrize("form", [None, "subpixel", "subscales", "radius4"])
@pytest.mark.parametrize("W,H,L", [(97, 65, 3), (160, 120, 3), (321, 243, 4), (513, 261, 5), (640, 485, 5)])
def test_tables_by_grid_size_leave_results_alone(form, W, H, L):
    kw = FORMS[form][0] if form else {}
    a, b = (torch.from_numpy(t).cuda() for t in frames(W, H, W))
    same(ff.flow_fields(a, b, ff.Params(levels=L, iters=3, **kw)),
         ff.flow_fields(a, b, ff.Params(levels=L, iters=3, tuning=ff.default_tuning(), **kw)))
