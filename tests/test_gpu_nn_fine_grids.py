"""NN search on seed grids so fine that the chunks' results do not fit the
scratch and are merged by atomics (and on both sides of that line), against the
squared distances of all pairs; and its time against the coarser grid's, whose
work per pixel pair is the same."""
import numpy as np
import pytest
import torch

import paper_1703_02563_amd as ff
from paper_1703_02563_amd.batch import BatchFlowFields

pytestmark = pytest.mark.gpu


def frames(W, H, seed, levels=256):
    g = torch.Generator().manual_seed(seed)
    return [torch.randint(0, levels, (H, W), generator=g).to(torch.uint8).cuda() for _ in range(2)]


def nearest(Da, Db, W, H, nc):
    """index and squared distance of the first nearest pixel of every cell"""
    q = Da[::nc, ::nc].reshape(-1, 16).float()
    r = Db.reshape(-1, 16).float()
    d = (q * q).sum(1)[:, None] + (r * r).sum(1)[None] - 2 * q @ r.T  # integers below 2^24: exact
    best = d.min(1).values
    return (d == best[:, None]).to(torch.uint8).argmax(1), best


@pytest.mark.parametrize("W,H,nc", [(96, 64, 1), (33, 200, 1), (97, 61, 2), (128, 96, 2), (160, 40, 4), (7, 5, 1),
                                    (64, 48, 8)])
@pytest.mark.parametrize("levels", [256, 3])
def test_search_on_fine_grids(W, H, nc, levels):
    a, b = frames(W, H, W + H + nc, levels)
    Da, Db = ff.descriptors(a, 1, rowmajor=True)[2], ff.descriptors(b, 1, rowmajor=True)[2]
    ca, cb = ff.descriptors(a, nc)[1], ff.descriptors(b, nc)[1]
    key = ff.init_nn(Da, Db, ca, cb, nc)[2].view(-1)
    idx, dist = nearest(Da, Db, W, H, nc)
    assert torch.equal(key & 0xFFFFFFFF, idx) and torch.equal(key >> 32, dist.long())


@pytest.mark.parametrize("levels", [1, 2])
def test_batch_on_fine_grids(levels):
    shapes = [(48, 64), (96, 128), (61, 97), (5, 300)]
    p = ff.Params(levels=levels, iters=2)
    batch = BatchFlowFields(shapes, p)
    pairs = [frames(W, H, W + H) for H, W in shapes]
    for k, (a, b) in enumerate(pairs):
        batch.set_pair(k, a, b)
    for o, (a, b) in zip(batch.run(), pairs):
        want = ff.flow_fields(a, b, p)
        for name, t in want.items():
            assert torch.equal(o[name], t), name


def test_one_direction_of_one_scale_uses_the_device():
    # every pixel a query: four times the pairs of a grid with a quarter of the queries
    def us(levels):
        a, b = frames(256, 192, 1)
        run = ff.FlowFields(256, 192, ff.Params(levels=levels, iters=1), backward=False)
        times = []
        for _ in range(6):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(20):
                run(a, b)
            e[1].record()
            e[1].synchronize()
            times.append(e[0].elapsed_time(e[1]) * 50)
        return min(times[1:])

    assert us(1) <= 2.5 * us(2)
