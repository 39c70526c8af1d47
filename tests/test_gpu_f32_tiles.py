"""Float-feature fields where the call gives no launch table: the tile of each
scale follows from its grid.  Sizes on both sides of each line, frames smaller
than a patch (every target clamped), odd sizes."""
import numpy as np
import pytest
import torch

import oracle
import paper_1703_02563_amd as ff
from paper_1703_02563_amd import learned as Lm
from test_learned_oracle import feature_canvas, feature_pyramid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,L", [
    (4, 5, 1), (7, 40, 2),   # no target 3n inside; a few at n = 1
    (57, 64, 3),             # 128 workgroups of 8x8 tiles at n = 1, fewer below
    (56, 64, 3),             # 112: 4x4
    (249, 250, 4),           # 512 workgroups of 16x16 tiles at n = 1
    (239, 250, 2),           # 480: 8x8
])
def test_fields_without_a_table_match_the_oracle(H, W, L):
    canvas = feature_canvas(H + W, H + 12, W + 12)
    F1 = canvas[6:6 + H, 6:6 + W].copy()
    F2 = canvas[3:3 + H, 8:8 + W].copy() + feature_canvas(5, H, W) * 0.05
    m1, m2 = feature_pyramid(F1, L), feature_pyramid(F2, L)
    prm = ff.Params(levels=L, iters=3)
    o = oracle.flow_fields_f32(m1, m2, L, 3, nthreads=8)
    g = Lm.flow_fields_f32([torch.from_numpy(a).cuda() for a in m1], [torch.from_numpy(a).cuda() for a in m2], prm)
    torch.cuda.synchronize()
    for k in ("flow_fwd", "flow_bwd", "keep_fwd", "keep_bwd"):
        assert np.array_equal(g[k].cpu().numpy(), o[k]), k
    for k in ("cost_fwd", "cost_bwd"):
        assert np.array_equal(g[k].cpu().numpy().view(np.uint32), o[k]), k
    assert tuple(int(v) for v in g["n_evals"].cpu()) == o["n_evals"]
