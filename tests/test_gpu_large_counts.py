"""Calls with more items than one launch takes: patch costs of more than 2^30
entries and split gradients of more than 2^30 pixels (four threads each), seed
candidates and their reranking on grids of
more than 2^20 cells (a wave each)."""
import pytest
import torch

import paper_1703_02563_amd as ff
from paper_1703_02563_amd import learned as Lm
from paper_1703_02563_amd.learned import cost_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def give_memory_back():
    yield
    torch.cuda.empty_cache()


def test_more_than_2_30_entries():
    count = (1 << 30) + 5
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB of device memory")
    W, H = 8, 4
    g = torch.Generator().manual_seed(0)
    f1, f2 = (torch.randn((H, W, 16), generator=g).cuda() for _ in range(2))
    entries = torch.zeros((count, 4), dtype=torch.int32, device="cuda")
    at = torch.tensor([0, 1, (1 << 29) - 1, 1 << 29, (1 << 29) + 1, (1 << 30) - 1, 1 << 30, count - 1], device="cuda")
    few = torch.stack([torch.arange(8) % W, torch.arange(8) % H, torch.zeros(8), torch.ones(8)], 1).int().cuda()
    entries[at] = few
    cost = cost_f32(f1, f2, entries, 1, 0)
    want = cost_f32(f1, f2, few, 1, 0)
    assert torch.equal(cost[at].view(torch.int32), want.view(torch.int32))
    zero = cost_f32(f1, f2, torch.zeros((1, 4), dtype=torch.int32, device="cuda"), 1, 0)
    rest = cost.view(torch.int32) != zero.view(torch.int32)
    rest[at] = False
    assert not bool(rest.any())


def test_more_than_2_30_pixels():
    pixels = (1 << 30) + 3
    if torch.cuda.mem_get_info()[0] < 150 << 30:
        pytest.skip("needs 150 GB of device memory")
    grad = torch.zeros((pixels, 16), device="cuda")
    at = torch.tensor([0, 1, (1 << 29) - 1, 1 << 29, (1 << 30) - 1, 1 << 30, pixels - 1], device="cuda")
    few = torch.randn((len(at), 16), generator=torch.Generator().manual_seed(0)).cuda()
    grad[at] = few
    hi, lo = (torch.full((pixels, 16), -1, dtype=torch.int16, device="cuda") for _ in range(2))
    ff.ffi.check(ff.lib().ff_l2norm16_bwd_split(None, None, Lm._ptr(grad), pixels, Lm._ptr(hi), Lm._ptr(lo),
                                                Lm._stream()), "ff_l2norm16_bwd_split")
    want = Lm._bf16_bits(few)
    assert torch.equal(hi[at], want) and torch.equal(lo[at], Lm._bf16_bits(few - Lm.bf16_bits_to_f32(want)))
    hi[at], lo[at] = 0, 0
    assert all(not bool(t.view(torch.int64).any()) for t in (hi, lo))


def test_more_than_2_20_cells():
    W, H, l, r = 1100, 1000, 3, 3
    g = torch.Generator(device="cuda").manual_seed(1)
    a, b = (torch.randint(0, 256, (H, W), generator=g, device="cuda").to(torch.uint8) for _ in range(2))
    (_, ma, Da), (_, mb, Db) = ff.descriptors(a, 1, rowmajor=True), ff.descriptors(b, 1, rowmajor=True)
    cand = ff.nn_topl(Da, Db, 1, l).view(-1, l)
    flow, cost, key = (t.reshape(H * W, -1) for t in ff.init_nn_l(Da, Db, ma, mb, 1, l, r))
    cells = torch.tensor([0, 1, (1 << 20) - 5, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 20) + 4099, W * H - 1],
                         device="cuda")
    dq, dr = Da.view(-1, 16).float(), Db.view(-1, 16).float()
    ys, xs = torch.arange(-r, r + 1, device="cuda"), torch.arange(-r, r + 1, device="cuda")
    for m in cells.tolist():
        d = (dr * dr).sum(1) - 2 * dr @ dq[m] + (dq[m] * dq[m]).sum()  # integers below 2^24: exact
        keys = (d.long() << 32) | torch.arange(W * H, device="cuda")
        want = keys.sort().values[:l]
        assert torch.equal(cand[m], want)

        def samples(D, i):
            y, x = (i // W + ys).clamp(0, H - 1), (i % W + xs).clamp(0, W - 1)
            return D[y][:, x].int()

        costs = [int((samples(Da, m) - samples(Db, int(q) & 0xFFFFFFFF)).abs().sum()) for q in want.tolist()]
        k = costs.index(min(costs))
        q = int(want[k]) & 0xFFFFFFFF
        assert int(key[m]) == int(want[k]) and int(cost[m]) == costs[k]
        assert flow[m].tolist() == [q % W - m % W, q // W - m // W]
