"""Workloads of the Flow Fields path that its speed is judged on.

Each case is one call (or one short pipeline) that a program using this
package makes: a frame pair through one of the schedules, a batch of pairs
of uneven sizes, the learned-descriptor path, the float patch cost with its
gradient, one training step.  All frames are synthetic: three-octave texture,
a moving background and star-shaped layers with motions up to 150 px, the
second frame with sensor noise.

Pair cases (path "pair") carry the schedule as plain values; a program keeps
a FlowFields runner (workspace and outputs) per frame size and passes new
frames to it.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1703_02563_amd as ff
from paper_1703_02563_amd import learned
from paper_1703_02563_amd.batch import BatchFlowFields

DEVICE = "cuda"

PLUS = {"iters": 8, "plus_iters": 4, "Rp": 2}  # 4 steps at R+ = 2R, then 8 at R on every scale


def listed():
    return [
        # the smallest frames (thumbnails, region crops): latency of one call
        {"name": "plain_160x120", "path": "pair", "W": 160, "H": 120, "levels": 3, "iters": 4},
        # the ordinary video frame pair, plain schedule, both fields and masks
        {"name": "plain_1024x436", "path": "pair", "W": 1024, "H": 436, "levels": 5, "iters": 6},
        # full-HD video, where the exact seed search grows with the square of the area
        {"name": "plain_1920x1080", "path": "pair", "W": 1920, "H": 1080, "levels": 6, "iters": 6},
        # the fast form on road-scene frames: no finest scale, one match per 2x2 region, R = 3/2
        {"name": "fast_x2_1242x375", "path": "pair", "W": 1242, "H": 375, "levels": 5, "R_num": 3, "R_den": 2,
         "fine_iters": 4, "fast_x2": True, **PLUS, "Rp": 6},
        # the accurate form with patch scales between the grid scales
        {"name": "subscales_1024x436", "path": "pair", "W": 1024, "H": 436, "levels": 5, "subscales": True, **PLUS},
        # the full matching pipeline: patch radius 4, two backward fields (radius 3), region filter, samples for
        # an interpolation step
        {"name": "filtered_r4_1024x436", "path": "filtered", "W": 1024, "H": 436, "levels": 5, "radius": 4,
         "radius2": 3, "s": 50, "q": 3, "e": 2, **PLUS},
        # flows in 1/8 px
        {"name": "subpixel_1024x436", "path": "pair", "W": 1024, "H": 436, "levels": 5, "iters": 6, "subpixel": 3},
        # eight seed candidates per cell, on an odd frame size
        {"name": "rerank8_741x497", "path": "pair", "W": 741, "H": 497, "levels": 5, "iters": 6, "nn_l": 8},
        # several pairs of uneven sizes per call (a serving loop; region proposals)
        {"name": "batch_8", "path": "batch", "pairs": 8, "shape_seed": 4, "levels": 5, "iters": 6},
        # the learned descriptor: network on every scale image, fields on its float features
        {"name": "learned_1024x436", "path": "learned", "W": 1024, "H": 436, "levels": 5, "iters": 6},
        # the float patch cost inside a user's own loss: forward and both gradients
        {"name": "patch_cost_1024x436", "path": "patch_cost", "W": 1024, "H": 436, "count": 65536, "n": 1,
         "radius": 3},
        # one optimiser step of the descriptor network on matches of the plain method
        {"name": "train_4x1024x436", "path": "train", "W": 1024, "H": 436, "pairs": 4, "samples": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _frame(rng, max_px, wmin=96, wmax=1920, hmin=64, hmax=1080):
    while True:
        W, H = _log_int(rng, wmin, wmax), _log_int(rng, hmin, hmax)
        if W * H <= max_px:
            return W, H


def _levels(rng, px):
    """Scales such that the coarsest grid keeps some hundred to some thousand cells, as the presets do."""
    if px < 60000:
        return rng.choice((3, 4))
    return rng.choice((4, 5)) if px < 300000 else rng.choice((5, 6)) if px > 700000 else 5


def draw(rng: random.Random):
    """A case of the same ranges: frames of 96x64 to full HD (the costlier forms up to 1024x436 pixels), any of
    the schedules."""
    kind = rng.choice(("plain", "plain", "plain", "fast", "fast", "subscales", "filtered", "subpixel", "rerank",
                       "batch", "learned", "patch_cost", "train"))
    if kind == "batch":
        return {"path": "batch", "pairs": rng.randint(2, 8), "shape_seed": rng.randint(1, 1 << 20), "levels": 5,
                "iters": rng.choice((4, 6))}
    if kind == "patch_cost":
        W, H = _frame(rng, 1024 * 436)
        return {"path": "patch_cost", "W": W, "H": H, "count": _log_int(rng, 512, 65536), "n": rng.choice((1, 1, 2, 4)),
                "radius": rng.choice((2, 3, 3, 4))}
    if kind == "train":
        W, H = _frame(rng, 1024 * 436, wmin=128, hmin=96)
        return {"path": "train", "W": W, "H": H, "pairs": rng.randint(1, 4), "samples": rng.choice((256, 512, 1024))}
    W, H = _frame(rng, 1920 * 1080 if kind == "plain" else 1024 * 436)
    c = {"path": "pair", "W": W, "H": H, "levels": _levels(rng, W * H), "iters": rng.choice((4, 6))}
    if kind == "plain":
        if rng.random() < 0.5:
            c.update(R_num=3, R_den=2)
    elif kind == "fast":  # Flow Fields+, Flow Fields+ Fast, Flow Fields+ Fast x2
        c.update(PLUS)
        form = rng.choice(("plus", "fast", "fast_x2"))
        if form != "plus":
            c.update(fine_iters=4)
        if form == "fast_x2":
            c.update(fast_x2=True)
    elif kind == "subscales":
        c.update(PLUS, subscales=True)
    elif kind == "filtered":
        r = rng.choice((3, 4))
        c.update(PLUS, path="filtered", radius=r, radius2=r - 1, s=50, q=rng.choice((3, 4)), e=2)
    elif kind == "subpixel":
        c.update(subpixel=3, nn_l=rng.choice((1, 4)))
    elif kind == "rerank":
        c.update(nn_l=rng.choice((2, 4, 8)))
    else:
        c.update(path="learned")
    return c


# --------------------------------------------------------------------------
# frames
# --------------------------------------------------------------------------

def _up(grid, s, H, W):
    y, x = torch.arange(H, device=DEVICE) / s, torch.arange(W, device=DEVICE) / s
    y0, x0 = y.long(), x.long()
    wy, wx = (y - y0)[:, None], (x - x0)[None, :]
    top = grid[y0][:, x0] * (1 - wx) + grid[y0][:, x0 + 1] * wx
    bot = grid[y0 + 1][:, x0] * (1 - wx) + grid[y0 + 1][:, x0 + 1] * wx
    return top * (1 - wy) + bot * wy


def _star(r, W, H, ys, xs):
    cx, cy, k = r.uniform(0, W), r.uniform(0, H), r.randint(3, 8)
    big = max(24.0, 0.45 * min(W, H))
    v = [(cx + d * math.cos(t), cy + d * math.sin(t))
         for t, d in zip(sorted(r.uniform(0, 2 * math.pi) for _ in range(k)), (r.uniform(0.1 * big, big) for _ in range(k)))]
    inside = torch.zeros((H, W), dtype=torch.bool, device=DEVICE)
    for (x1, y1), (x2, y2) in zip(v, v[1:] + v[:1]):
        if y1 != y2:
            inside ^= ((y1 > ys) != (y2 > ys)) & (xs < (x2 - x1) * (ys - y1) / (y2 - y1) + x1)
    return inside


def _pair(W, H, seed):
    """Two uint8 frames [H][W]: texture layers at integer displacements."""
    r = random.Random(seed)
    g = torch.Generator(device=DEVICE).manual_seed(r.getrandbits(40))
    t_max = max(4, min(150, min(W, H) // 3))
    pad = t_max + 66
    ch, cw = H + 2 * pad, W + 2 * pad
    canvas = torch.rand((ch, cw), generator=g, device=DEVICE)
    for s in (4, 16):
        canvas += _up(torch.rand((ch // s + 2, cw // s + 2), generator=g, device=DEVICE), s, ch, cw)
    canvas = canvas * (255.0 / 3.0)
    ys, xs = torch.arange(H, device=DEVICE)[:, None], torch.arange(W, device=DEVICE)[None, :]
    b = max(1, t_max // 5)
    tx, ty = r.randint(-b, b), r.randint(-b, b)
    img1 = canvas[pad:pad + H, pad:pad + W].clone()
    img2 = canvas[pad - ty:pad - ty + H, pad - tx:pad - tx + W].clone()
    for _ in range(12):
        m = _star(r, W, H, ys.float(), xs.float())
        tx, ty, ox, oy = r.randint(-t_max, t_max), r.randint(-t_max, t_max), r.randint(-64, 64), r.randint(-64, 64)
        img1 = torch.where(m, canvas[pad + oy:pad + oy + H, pad + ox:pad + ox + W], img1)
        m2 = torch.zeros_like(m)
        m2[max(0, ty):H + min(0, ty), max(0, tx):W + min(0, tx)] = \
            m[max(0, -ty):H + min(0, -ty), max(0, -tx):W + min(0, -tx)]
        src = canvas[pad + oy - ty:pad + oy - ty + H, pad + ox - tx:pad + ox - tx + W]
        img2 = torch.where(m2, src, img2)
    img2 = img2 + 2.0 * torch.randn((H, W), generator=g, device=DEVICE)
    return tuple(t.round().clamp(0, 255).to(torch.uint8).contiguous() for t in (img1, img2))


def _params(c):
    return ff.Params(levels=c["levels"], iters=c["iters"], radius=c.get("radius", 3), R_num=c.get("R_num", 1),
                     R_den=c.get("R_den", 1), plus_iters=c.get("plus_iters", 0), Rp_num=c.get("Rp", 0),
                     fine_iters=c.get("fine_iters", 0), subpixel=c.get("subpixel", 0), nn_l=c.get("nn_l", 1),
                     fast_x2=c.get("fast_x2", False), subscales=c.get("subscales", False))


def _batch_shapes(c):
    r = random.Random(c["shape_seed"])
    return [(r.randint(192, 512), r.randint(256, 1280)) for _ in range(c["pairs"])]


# --------------------------------------------------------------------------
# the passes
# --------------------------------------------------------------------------

def _patch_cost_inputs(case, seed):
    """Unit-length features of two frames, matches with small errors around a common motion, upstream gradient."""
    W, H, m = case["W"], case["H"], case["count"]
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    f1 = torch.nn.functional.normalize(torch.randn((H, W, 16), generator=g, device=DEVICE), dim=2)
    f2 = torch.nn.functional.normalize(torch.roll(f1, (3, -5), (0, 1))
                                       + 0.1 * torch.randn((H, W, 16), generator=g, device=DEVICE), dim=2)
    x = torch.randint(0, W, (m,), generator=g, device=DEVICE)
    y = torch.randint(0, H, (m,), generator=g, device=DEVICE)
    o = torch.randint(-8, 9, (m, 2), generator=g, device=DEVICE)
    tx, ty = (x - 5 + o[:, 0]).clamp(0, W - 1), (y + 3 + o[:, 1]).clamp(0, H - 1)
    entries = torch.stack([x, y, tx - x, ty - y], 1).to(torch.int32).contiguous()
    return f1.contiguous(), f2.contiguous(), entries, torch.randn(m, generator=g, device=DEVICE) / m


def prepare(case, seed):
    path = case["path"]
    if path == "pair":
        i1, i2 = _pair(case["W"], case["H"], seed)
        return {"path": path, "i1": i1, "i2": i2, "runner": ff.FlowFields(case["W"], case["H"], _params(case))}
    if path == "filtered":
        i1, i2 = _pair(case["W"], case["H"], seed)
        return {"path": path, "i1": i1, "i2": i2, "params": _params(case), "case": dict(case)}
    if path == "batch":
        b = BatchFlowFields(_batch_shapes(case), _params(case))
        for k, (H, W) in enumerate(b.shapes):
            b.set_pair(k, *_pair(W, H, seed * 64 + k))
        return {"path": path, "batch": b}
    if path == "learned":
        i1, i2 = _pair(case["W"], case["H"], seed)
        return {"path": path, "i1": i1, "i2": i2, "params": _params(case), "net": learned.DescNet(seed=seed % 1000)}
    if path == "patch_cost":
        f1, f2, entries, g = _patch_cost_inputs(case, seed)
        return {"path": path, "f1": f1.requires_grad_(), "f2": f2.requires_grad_(), "entries": entries, "grad": g,
                "case": dict(case)}
    items = []  # training pairs with the plain method's matches
    for k in range(case["pairs"]):
        i1, i2 = _pair(case["W"], case["H"], seed * 64 + k)
        o = ff.flow_fields(i1, i2, ff.Params(levels=5, iters=6))
        items.append((i1, i2, learned.TripletSampler(o["flow_fwd"], o["keep_fwd"])))
    return {"path": path, "net": learned.DescNet(seed=seed % 1000), "items": items,
            "rng": np.random.default_rng(seed), "samples": case["samples"]}


def run(state):
    path = state["path"]
    if path == "pair":
        return state["runner"](state["i1"], state["i2"])
    if path == "filtered":
        c = state["case"]
        o = ff.flow_fields_two_backward(state["i1"], state["i2"], state["params"], radius2=c["radius2"])
        keep = ff.region_filter(o["flow_fwd"], o["cost_fwd"], o["keep_fwd"], c["s"])
        sel = ff.sparsify(o["flow_fwd"], keep, o["flow_bwd"], o["flow_bwd2"], c["q"], c["e"])
        return dict(o, filtered=keep, selection=sel)
    if path == "batch":
        return state["batch"].run()
    if path == "learned":
        return learned.learned_flow_fields(state["net"], state["i1"], state["i2"], state["params"])
    if path == "patch_cost":
        c = state["case"]
        cost = learned.patch_cost(state["f1"], state["f2"], state["entries"], c["n"], c["radius"])
        g1, g2 = torch.autograd.grad(cost, (state["f1"], state["f2"]), state["grad"])
        return {"cost": cost.detach(), "g1": g1, "g2": g2}
    loss = learned.train_step(state["net"], state["items"], state["rng"], samples=state["samples"])
    return {"loss": loss, "w": list(state["net"].w), "b": list(state["net"].b)}


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def _cells(W, H, n):
    return -(-W // n) * -(-H // n)


def _fields_work(c, W, H, directions=2, sample_ops=3, samples=None):
    """Frames in, fields and masks out; the exact seed search (16 products per cell and pixel), and per cell and
    scale about two propagation evaluations plus one per random search, each over the (2r + 7)^2 distinct samples
    of a patch."""
    px, L = W * H, c["levels"]
    fast2 = bool(c.get("fast_x2"))
    scales = [1 << k for k in range(1 if fast2 else 0, L)]
    out = _cells(W, H, 2) if fast2 else px
    T, P = c["iters"], c.get("plus_iters", 0)
    samples = samples or (2 * c.get("radius", 3) + 7) ** 2
    searches = (T - 1) + max(0, P - 1)
    evals = 0
    for n in scales:
        stages = 2 if c.get("subscales") and 1 < n < (1 << (L - 1)) else 1
        rs = c["fine_iters"] - 1 if c.get("fine_iters") and n == scales[0] else searches
        evals += stages * _cells(W, H, n) * (2 + rs)
    refs = _cells(W, H, 2) if fast2 else px
    seed_ops = 32 * _cells(W, H, scales[-1]) * refs
    return {"bytes": 2 * px + directions * out * 9, "flops": directions * (seed_ops + evals * samples * sample_ops)}


def work(case):
    path = case["path"]
    if path == "batch":
        w = [_fields_work(case, W, H) for H, W in _batch_shapes(case)]
        return {k: sum(v[k] for v in w) for k in ("bytes", "flops")}
    W, H = case["W"], case["H"]
    px = W * H
    if path == "pair":
        return _fields_work(case, W, H)
    if path == "filtered":
        a = _fields_work(case, W, H)
        b = _fields_work(dict(case, radius=case["radius2"]), W, H, directions=1)
        return {"bytes": a["bytes"] + px * 8 + px + 4 * _cells(W, H, case["q"]), "flops": a["flops"] + b["flops"]}
    if path == "learned":
        a = _fields_work(case, W, H, samples=784)
        return {"bytes": a["bytes"], "flops": a["flops"] + 2 * case["levels"] * px * 28224}
    if path == "patch_cost":
        m, k = case["count"], (2 * case["radius"] + 1) ** 2 * 16
        return {"bytes": 4 * 64 * px + 24 * m, "flops": m * k * 7}  # 3 forward; 4 for the two gradients
    B, m = case["pairs"], case["samples"]
    # the images in; forward, data and weight gradients of the network (28224 forward, twice that backward less
    # the first layer's data gradient), both patch costs with their gradients
    return {"bytes": 2 * B * px, "flops": 2 * B * px * (3 * 28224 - 576) + B * 2 * m * 784 * 7}


# --------------------------------------------------------------------------
# 64-bit values
# --------------------------------------------------------------------------

def exact(case, seed):
    """Only the float patch cost has one: every other output is whole numbers (fields, masks, counts, costs and
    float bit patterns), or a training step of a network defined by its bf16 roundings."""
    if case["path"] != "patch_cost":
        return None
    f1, f2, entries, g = _patch_cost_inputs(case, seed)
    f1, f2, g = f1.double(), f2.double(), g.double()
    W, H, n, r = case["W"], case["H"], case["n"], case["radius"]
    x, y, fx, fy = (entries[:, k].long() for k in range(4))
    cost = torch.zeros(case["count"], dtype=torch.float64, device=DEVICE)
    g1, g2 = (torch.zeros((H * W, 16), dtype=torch.float64, device=DEVICE) for _ in range(2))
    for v in range(-r, r + 1):
        for u in range(-r, r + 1):
            p = (y + n * v).clamp(0, H - 1) * W + (x + n * u).clamp(0, W - 1)
            q = (y + fy + n * v).clamp(0, H - 1) * W + (x + fx + n * u).clamp(0, W - 1)
            d = f1.view(-1, 16)[p] - f2.view(-1, 16)[q]
            cost += (d * d).sum(1)
            d = 2 * g[:, None] * d
            g1.index_add_(0, p, d)
            g2.index_add_(0, q, -d)
    return {"cost": cost, "g1": g1.view(H, W, 16), "g2": g2.view(H, W, 16)}
