"""NN search and l nearest references at the sizes where their tiling can go
wrong (query blocks per wave, chunk and group ends, the atomic merge of
one-pixel grids, ties and full candidate lists), bit-exact against distances
computed in float64 (exact: every distance is below 2^21)."""
import numpy as np
import pytest
import torch

import paper_1703_02563_amd as ff

pytestmark = pytest.mark.gpu


def nearest(Da, Db, nc, l, rows):
    """(distance << 32) | q of the l nearest pixels of the sampled cells."""
    H, W, _ = Da.shape
    q = Da[::nc, ::nc].reshape(-1, 16).double()[rows]
    b = Db.reshape(-1, 16).double()
    d = ((q * q).sum(1)[:, None] + (b * b).sum(1)[None] - 2 * q @ b.T).round().long()
    key = (d << 32) | torch.arange(W * H, device="cuda")[None]
    k = min(l, W * H)
    out = torch.full((len(rows), l), -1, dtype=torch.int64, device="cuda")
    out[:, :k] = key.topk(k, dim=1, largest=False, sorted=True).values
    return out


def descs(W, H, kind, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if kind == "flat":    # every reference ties
        return torch.full((H, W, 16), 77, dtype=torch.uint8, device="cuda")
    hi = 2 if kind == "two" else 256
    d = torch.randint(0, hi, (H, W, 16), generator=g, device="cuda").to(torch.uint8)
    if kind == "extreme":  # the largest distances: 0 against 255
        d = torch.where(d < 128, 0, 255).to(torch.uint8)
    if kind == "flat_far":  # large near-tied areas of which only a few pixels are nearest
        d = (d < 3).to(torch.uint8) * 5
    return d


@pytest.mark.parametrize("W,H,nc,kind", [
    (1, 1, 1, "noise"), (33, 7, 16, "noise"), (5, 3, 2, "noise"),          # fewer references than a tile, or than l
    (64, 48, 4, "noise"), (64, 64, 4, "two"), (65, 64, 4, "noise"),        # 192, 256, 272 queries
    (128, 64, 4, "noise"), (129, 64, 4, "flat"), (130, 67, 2, "two"),      # 512, 528 queries
    (70, 50, 1, "extreme"), (400, 330, 1, "noise"),                        # one-pixel grids: the second merges by atomics
    (643, 480, 16, "flat"), (643, 481, 32, "flat_far"),
])
def test_nearest_and_l_nearest(W, H, nc, kind):
    Da, Db = descs(W, H, "noise" if kind == "flat_far" else kind, 1), descs(W, H, kind, 2)
    mc = torch.zeros((H + 8 * nc, W + 8 * nc, 16), dtype=torch.uint8, device="cuda")
    _, _, key = ff.init_nn(Da, Db, mc, mc, nc, 0)
    M = key.numel()
    rows = torch.arange(M, device="cuda") if M <= 600 else torch.linspace(0, M - 1, 600, device="cuda").long()
    assert torch.equal(key.view(-1)[rows], nearest(Da, Db, nc, 1, rows)[:, 0])
    if W * H > 100000 and nc == 1:
        return
    for l in (1, 3, 8):
        got = ff.nn_topl(Da, Db, nc, l).view(M, l)[rows]
        assert torch.equal(got, nearest(Da, Db, nc, l, rows)), l
