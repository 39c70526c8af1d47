"""The folded passes of a training step against the passes they fold, at the
sizes where their tiles, columns of 16 pixels and runs of rows end."""
import numpy as np
import pytest
import torch

import paper_1703_02563_amd as ff
from paper_1703_02563_amd import learned as Lm

pytestmark = pytest.mark.gpu
P, S = Lm._ptr, Lm._stream
SIZES = [(1, 1, 1), (2, 5, 3), (1, 9, 16), (1, 3, 17), (3, 8, 33), (2, 37, 61), (5, 64, 47)]


def call(name, *args):
    ff.ffi.check(getattr(ff.lib(), name)(*args, S()), name)


def bf16(shape, g, scale=1.0):
    return Lm._bf16_bits((torch.randn(shape, generator=g) * scale).cuda())


def split(x):
    hi = Lm._bf16_bits(x)
    return hi, Lm._bf16_bits(x - Lm.bf16_bits_to_f32(hi))


@pytest.mark.parametrize("B,H,W", SIZES)
def test_last_layer_with_normalisation(B, H, W):
    g = torch.Generator().manual_seed(B * H + W)
    x, w, b = bf16((B, H, W, 32), g), bf16((16, 9, 32), g, 0.1), torch.randn(16, generator=g).cuda()
    want, inv = torch.empty((B, H, W, 16), device="cuda"), torch.empty((B, H, W), device="cuda")
    call("ff_conv3x3_fwd", P(x), B, H, W, 32, 16, P(w), P(b), 0, P(want), None)
    call("ff_l2norm16_fwd", P(want), B * H * W, 1e-4, P(want), P(inv))
    got, ginv = torch.empty_like(want), torch.empty_like(inv)
    call("ff_conv3x3_norm_fwd", P(x), B, H, W, P(w), P(b), 1e-4, P(got), P(ginv))
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    assert torch.equal(ginv.view(torch.int32), inv.view(torch.int32))


@pytest.mark.parametrize("cout", [16, 32])
@pytest.mark.parametrize("B,H,W", SIZES)
def test_data_gradient_through_relu_split(B, H, W, cout):
    g = torch.Generator().manual_seed(B * H + W + cout)
    go, w = bf16((B, H, W, cout), g), bf16((cout, 9, 32), g, 0.1)
    act = bf16((B, H, W, 32), g).clamp(min=0)  # negative bf16 have a negative bit pattern
    flip = torch.empty((32, 9, cout), dtype=torch.int16, device="cuda")
    gin = torch.empty((B, H, W, 32), device="cuda")
    call("ff_conv3x3_bwd_data", P(go), B, H, W, 32, cout, P(w), P(flip), P(gin), None)
    call("ff_relu_bwd", P(act), P(gin), gin.numel(), P(gin), None)
    hi, lo = (torch.empty((B, H, W, 32), dtype=torch.int16, device="cuda") for _ in range(2))
    call("ff_conv3x3_bwd_data_split", P(go), B, H, W, 32, cout, P(w), P(flip), P(act), P(hi), P(lo))
    for a, b in zip((hi, lo), split(gin)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("with_norm", [True, False])
@pytest.mark.parametrize("pixels", [1, 3, 63, 65, 1000])
def test_normalisation_gradient_split(pixels, with_norm):
    g = torch.Generator().manual_seed(pixels)
    y, go = (torch.randn((pixels, 16), generator=g).cuda() for _ in range(2))
    inv = torch.rand(pixels, generator=g).cuda()
    want = go.clone()
    if with_norm:
        call("ff_l2norm16_bwd", P(y), P(inv), P(go), pixels, P(want))
    hi, lo = (torch.empty((pixels, 16), dtype=torch.int16, device="cuda") for _ in range(2))
    call("ff_l2norm16_bwd_split", P(y) if with_norm else None, P(inv) if with_norm else None, P(go), pixels, P(hi),
         P(lo))
    for a, b in zip((hi, lo), split(want)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("cin,cout", [(1, 32), (32, 32), (32, 16)])
@pytest.mark.parametrize("B,H,W", SIZES + [(2, 200, 40)])
def test_weight_gradient_both_forms(cin, cout, B, H, W):
    """The same bits from a float32 gradient and from its two parts, and within
    the float32 accumulation bound of the parts' gradient in float64."""
    g = torch.Generator().manual_seed(B * H + W + cin + cout)
    x = bf16((B, H, W, cin), g)
    go = torch.randn((B, H, W, cout), generator=g).cuda()
    nbytes = int(ff.lib().ff_conv3x3_wgrad_scratch_bytes(B, H, cin, cout))
    scratch = torch.full((nbytes // 4,), float("nan"), device="cuda")
    out = []
    for form in range(2):
        gw, gb = torch.empty((cout, 9, cin), device="cuda"), torch.empty(cout, device="cuda")
        if form == 0:
            call("ff_conv3x3_bwd_weight", P(x), P(go), B, H, W, cin, cout, P(scratch), nbytes, P(gw), P(gb))
        else:
            hi, lo = split(go)
            call("ff_conv3x3_bwd_weight_split", P(x), P(hi), P(lo), B, H, W, cin, cout, P(scratch), nbytes, P(gw),
                 P(gb))
        out.append((gw, gb))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    xf = np.pad(Lm.bf16_bits_to_f32(x).double().cpu().numpy(), ((0, 0), (1, 1), (1, 1), (0, 0)))
    gf = sum(Lm.bf16_bits_to_f32(t).double() for t in split(go)).cpu().numpy().reshape(-1, cout)
    bound = 3.1 * B * H * W * 2.0 ** -24
    for tap in range(9):
        xt = xf[:, tap // 3:tap // 3 + H, tap % 3:tap % 3 + W].reshape(-1, cin)
        err = np.abs(out[0][0][:, tap].double().cpu().numpy() - gf.T @ xt)
        assert np.all(err <= bound * (np.abs(gf).T @ np.abs(xt)) + 1e-30), tap
    assert np.all(np.abs(out[0][1].double().cpu().numpy() - gf.sum(0)) <= bound * np.abs(gf).sum(0))
