"""Outputs of the 3x3 convolutions: float32 and bf16, aligned for 16-byte stores
and to an element only, around the ends of their tiles (32 pixels, 8 rows) and
of the runs of tiles that a workgroup takes (more of them from 256, 512 and 768
tiles on); and calls that have to stay as quick as others that move the same
bytes."""
import pytest
import torch

import paper_1703_02563_amd as ff
from paper_1703_02563_amd import learned as Lm

pytestmark = pytest.mark.gpu
P, S = Lm._ptr, Lm._stream


def call(name, *args):
    ff.ffi.check(getattr(ff.lib(), name)(*args, S()), name)


def bf16(shape, g, scale=1.0):
    return Lm._bf16_bits((torch.randn(shape, generator=g) * scale).cuda())


def outputs(n, off):
    """float32 and bf16 buffers of n values, `off` values past a 16-byte boundary, and a guard behind them"""
    f, h = torch.full((n + off + 8,), -7.0, device="cuda"), torch.full((n + off + 8,), -7, dtype=torch.int16, device="cuda")
    return f, h, f[off:off + n], h[off:off + n]


@pytest.mark.parametrize("cin,cout", [(1, 32), (32, 32), (32, 16), (16, 32)])
@pytest.mark.parametrize("B,H,W", [(1, 1, 1), (2, 8, 32), (1, 9, 33), (3, 33, 31), (1, 2049, 5), (1, 4100, 3),
                                   (1, 6150, 2), (2, 17, 1100)])
def test_outputs_of_every_kind(B, H, W, cin, cout):
    g = torch.Generator().manual_seed(B * H + W + cin)
    x, w, b = bf16((B, H, W, cin), g), bf16((cout, 9, cin), g, 0.1), torch.randn(cout, generator=g).cuda()
    n = B * H * W * cout
    xd = Lm.bf16_bits_to_f32(x).double().permute(0, 3, 1, 2)
    wd = Lm.bf16_bits_to_f32(w).double().view(cout, 3, 3, cin).permute(0, 3, 1, 2)
    unfold = torch.nn.functional.unfold  # (products by a plain matrix product in 64 bits)
    cols = unfold(xd, 3, padding=1)
    wm = wd.reshape(cout, -1)
    want = (wm @ cols + b.double()[:, None]).permute(0, 2, 1).reshape(-1)
    mass = (wm.abs() @ cols.abs() + b.double().abs()[:, None]).permute(0, 2, 1).reshape(-1)
    first = None
    for off in (0, 1):
        fa, ha, f, h = outputs(n, off)
        call("ff_conv3x3_fwd", P(x), B, H, W, cin, cout, P(w), P(b), 0, P(f), P(h))
        # at most 9 cin + 1 additions, each within 2^-24 of the sum of magnitudes
        assert bool(((f.double() - want).abs() <= (9 * cin + 1) * 2.0 ** -24 * mass).all())
        assert torch.equal(h, Lm._bf16_bits(f))
        for whole, pad in ((fa, -7.0), (ha, -7)):
            assert bool((whole[:off] == pad).all()) and bool((whole[off + n:] == pad).all())
        if off == 0:
            first = f.clone()
        assert torch.equal(f.view(torch.int32), first.view(torch.int32))
        fa, ha, f2, h2 = outputs(n, off)  # one output alone, with ReLU
        call("ff_conv3x3_fwd", P(x), B, H, W, cin, cout, P(w), P(b), 1, P(f2), None)
        call("ff_conv3x3_fwd", P(x), B, H, W, cin, cout, P(w), P(b), 1, None, P(h2))
        assert torch.equal(f2, f.clamp(min=0)) and torch.equal(h2, Lm._bf16_bits(f.clamp(min=0)))


def launch_us(fn, launches=40):
    """us a launch inside a graph of `launches`, the best of five replays"""
    fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(launches):
            fn()
    times = []
    for _ in range(6):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / launches)
    return min(times[1:])


def conv_us(B, H, W, cin, cout, f32):
    g = torch.Generator().manual_seed(1)
    x, w, b = bf16((B, H, W, cin), g), bf16((cout, 9, cin), g, 0.1), torch.zeros(cout).cuda()
    out = torch.empty((B, H, W, cout), dtype=torch.float32 if f32 else torch.int16, device="cuda")
    return launch_us(lambda: call("ff_conv3x3_fwd", P(x), B, H, W, cin, cout, P(w), P(b), 0, P(out) if f32 else None,
                                  None if f32 else P(out)))


def test_float_outputs_cost_their_bytes():
    # 64 bytes a pixel read and 64 (bf16) or 128 (float32) written: 1.5 times the bytes
    assert conv_us(2, 480, 640, 32, 32, True) <= 1.75 * conv_us(2, 480, 640, 32, 32, False)


@pytest.mark.parametrize("cin,cout", [(32, 32), (32, 16)])
def test_a_few_tiles_run_side_by_side(cin, cout):
    # 16 tiles as four rows of four, and one tile: not one after another
    assert conv_us(1, 32, 128, cin, cout, False) <= 1.3 * conv_us(1, 8, 32, cin, cout, False)


@pytest.mark.parametrize("cin,cout", [(32, 32), (32, 16)])
def test_weight_gradient_of_a_small_image_runs_side_by_side(cin, cout):
    def us(B, H, W):
        g = torch.Generator().manual_seed(1)
        x, go = bf16((B, H, W, cin), g), torch.randn((B, H, W, cout), generator=g).cuda()
        nbytes = int(ff.lib().ff_conv3x3_wgrad_scratch_bytes(B, H, cin, cout))
        scratch = torch.empty(nbytes // 4, device="cuda")
        gw, gb = torch.empty(cout * 9 * cin, device="cuda"), torch.empty(cout, device="cuda")
        return launch_us(lambda: call("ff_conv3x3_bwd_weight", P(x), P(go), B, H, W, cin, cout, P(scratch), nbytes,
                                      P(gw), P(gb)))

    # 16 rows of one column of 16 pixels against eight times as many
    assert us(1, 32, 64) <= 1.5 * us(1, 16, 16)
