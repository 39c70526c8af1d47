"""Scales of a single cell, whose launches take as many steps as the widest halo
holds: the fields, costs and counts of a call are those under the built-in table
of a larger frame."""
import pytest
import torch

import paper_1703_02563_amd as ff

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,kw", [
    (64, 48, dict(levels=7, iters=12)), (33, 20, dict(levels=7, iters=4)), (64, 64, dict(levels=7, iters=7, nn_l=4)),
    (40, 30, dict(levels=7, iters=6, subpixel=3)), (40, 30, dict(levels=7, iters=5, radius=2)),
    (40, 30, dict(levels=7, iters=5, radius=4)), (40, 30, dict(levels=7, iters=5, subscales=True)),
    (20, 20, dict(levels=6, iters=6, plus_iters=4, Rp_num=2)), (32, 17, dict(levels=6, iters=6, fast_x2=True)),
])
def test_fields_do_not_depend_on_the_tables(W, H, kw):
    g = torch.Generator().manual_seed(W + H)
    a, b = (torch.randint(0, 256, (H, W), generator=g).to(torch.uint8).cuda() for _ in range(2))
    got, want = (ff.flow_fields(a, b, ff.Params(tuning=t, **kw)) for t in (None, ff.default_tuning()))
    for name in want:
        assert torch.equal(got[name], want[name]), name
