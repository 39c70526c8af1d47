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
