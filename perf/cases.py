"""The work that a user of this library has it do, as cases that can be timed.

A camera or photo pipeline registers pairs and stacks of exposures and merges
them; a service registers many uneven pairs at once; a tool calls one stage
(search, propagation, warp, merge) on images of its own; the learned proposal
is evaluated and trained. listed() holds one case of each, draw() more cases of
the same ranges.

Inputs are synthetic exposure stacks made on the GPU from the seed: smooth
structure at three scales plus pixel texture, seen through a homography and
per-tile integer shifts, scaled by the exposure ratio, with sensor noise.
"""
import math
import random

import numpy as np
import torch
import torch.nn.functional as F

import paper_1504_01441_amd as lnr
from paper_1504_01441_amd import proposal

TILE = 32
LARGEST = (4032, 3024)   # the largest frame of the ranges
_CTX = None


def listed():
    return [
        # A preview-sized luma pair, where latency and launches count.
        dict(name="pair_vga_y8", kind="pair", width=640, height=480, format="y8", radius=8,
             ratio=4.0, learned=False),
        # A phone's still: one 5 MP colour pair, the benchmark's registration.
        dict(name="pair_5mp_i420", kind="pair", width=2592, height=1944, format="i420", radius=16,
             ratio=8.0, learned=False),
        # The same with the learned proposal narrowing the level-0 search.
        dict(name="pair_5mp_learned", kind="pair", width=2592, height=1944, format="i420",
             radius=16, ratio=8.0, learned=True),
        # A full-resolution bracket: three 12 MP frames to the shortest one.
        dict(name="stack_12mp_3", kind="stack", width=4000, height=3000, format="i420", radius=16,
             frames=3),
        # A service's queue: uneven pairs in one call.
        dict(name="batch_8_uneven", kind="batch", pairs=8, sizes=7, max_width=1920,
             max_height=1440, radius=16),
        # The matcher alone on a warped frame.
        dict(name="search_3mp", kind="search", width=2048, height=1536, radius=16),
        # Sparse matches to a dense flow at an odd size.
        dict(name="flow_8mp_odd", kind="flow", width=3263, height=2447),
        # Backward warp of an interleaved-chroma frame.
        dict(name="warp_5mp_nv12", kind="warp", width=2592, height=1944, format="nv12"),
        # Deghosted fusion of a registered 5 MP pair, the benchmark's merge.
        dict(name="merge_5mp_2", kind="merge", width=2592, height=1944, format="i420", frames=2),
        # Irradiance map of a registered three-frame stack at a video-like size.
        dict(name="irradiance_1mp_3", kind="irradiance", width=1280, height=960, format="nv12",
             frames=3),
        # The proposal network over every tile of a 5 MP frame.
        dict(name="network_forward", kind="forward", tiles=4860),
        # One training step at the training pipeline's batch size.
        dict(name="network_train", kind="train", tiles=256),
    ]


def draw(rng):
    kind = rng.choice(["pair", "pair", "pair", "stack", "batch", "search", "flow", "flow", "warp",
                       "merge", "merge", "irradiance", "forward", "train"])
    fmt = rng.choice(["y8", "i420", "nv12"])
    if kind == "forward":
        return dict(kind=kind, tiles=int(round(math.exp(rng.uniform(math.log(40), math.log(11000))))))
    if kind == "train":
        return dict(kind=kind, tiles=int(round(math.exp(rng.uniform(math.log(32), math.log(1024))))))
    if kind == "batch":
        return dict(kind=kind, pairs=rng.randint(3, 12), sizes=rng.randrange(1 << 20),
                    max_width=2 * rng.randint(400, 1000), max_height=2 * rng.randint(300, 750),
                    radius=rng.choice([8, 12, 16]))
    most = {"stack": 8e6, "merge": 8e6}.get(kind, float(LARGEST[0] * LARGEST[1]))
    area = math.exp(rng.uniform(math.log(320 * 240), math.log(most)))
    aspect = rng.uniform(1.0, 1.8)
    w = min(LARGEST[0], max(160, int(round(math.sqrt(area * aspect)))))
    h = min(LARGEST[1], max(160, int(round(math.sqrt(area / aspect)))))
    if rng.random() < 0.25:
        w, h = min(h, LARGEST[0]), min(w, LARGEST[1])
    if fmt != "y8":
        w, h = w // 2 * 2, h // 2 * 2
    c = dict(kind=kind, width=w, height=h)
    if kind in ("pair", "stack", "warp", "merge", "irradiance"):
        c["format"] = fmt
    if kind in ("pair", "stack", "search"):
        c["radius"] = rng.choice([8, 10, 12, 16, 16, 24])
    if kind == "pair":
        c["ratio"] = round(rng.uniform(2.0, 16.0), 2)
        c["learned"] = rng.random() < 0.25
    if kind in ("stack", "merge", "irradiance"):
        c["frames"] = rng.choice([2, 3, 3, 4]) if kind != "stack" else rng.choice([2, 3])
    return c


# ----------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda")


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _smooth(g, h, w, cell, amp):
    """Smooth random field in [-amp, amp] with features about `cell` wide."""
    gh, gw = max(4, int(h / cell) + 3), max(4, int(w / cell) + 3)
    f = 2.0 * _rand(g, 1, 1, gh, gw) - 1.0
    return amp * F.interpolate(f, size=(h, w), mode="bicubic", align_corners=True)[0, 0]


def _sample(img, x, y):
    """Bilinear samples of img at float positions, clamped to the edge."""
    h, w = img.shape
    x, y = x.clamp(0, w - 1), y.clamp(0, h - 1)
    x0, y0 = x.floor().clamp(max=max(w - 2, 0)), y.floor().clamp(max=max(h - 2, 0))
    ax, ay = x - x0, y - y0
    i = y0.long() * w + x0.long()
    f = img.reshape(-1)
    dx, dy = (1 if w > 1 else 0), (w if h > 1 else 0)
    return ((1 - ay) * ((1 - ax) * f[i] + ax * f[i + dx])
            + ay * ((1 - ax) * f[i + dy] + ax * f[i + dy + dx]))


def _homography(rng, w, h, max_rot_deg=2.0, max_trans=10.0, max_persp=1e-4):
    th = math.radians(rng.uniform(-max_rot_deg, max_rot_deg))
    p = max_persp * 640.0 / w
    a = np.array([[math.cos(th), -math.sin(th), rng.uniform(-max_trans, max_trans)],
                  [math.sin(th), math.cos(th), rng.uniform(-max_trans, max_trans)],
                  [rng.uniform(-p, p), rng.uniform(-p, p), 1.0]])
    t = np.array([[1, 0, (w - 1) / 2.0], [0, 1, (h - 1) / 2.0], [0, 0, 1.0]])
    return t @ a @ np.linalg.inv(t)


def _u8(x):
    return x.round().clamp(0, 255).to(torch.uint8)


def _frames(w, h, seed, ratios, fmt, shift=6, movers=0.1, saturated=0.0):
    """Exposures of one scene as library frames; the first is the reference geometry."""
    g, rng = _gen(seed), random.Random(seed)
    m = int(64 + 0.06 * max(w, h))
    ch, cw = h + 2 * m, w + 2 * m
    scene = (_smooth(g, ch, cw, w / 6, 40.0) + _smooth(g, ch, cw, w / 20, 25.0)
             + _smooth(g, ch, cw, max(w / 80, 6.0), 12.0) + 16.0 * _rand(g, ch, cw) - 8.0)
    scene += 120.0 / ratios[1] - scene[m:m + h, m:m + w].median()
    if saturated > 0:
        f = _smooth(g, ch, cw, w / 12, 1.0)
        n = f.numel()
        level = f.reshape(-1)[:: max(1, n // 1000000)].sort().values
        scene = torch.where(f > level[int((1 - saturated) * level.numel())],
                            torch.full_like(scene, 1e4), scene)
    chroma = [128.0 + _smooth(g, ch, cw, w / 10, 24.0) for _ in range(2)] if fmt != "y8" else None
    ty, tx = max(h // TILE, 1), max(w // TILE, 1)
    out = []
    for k, ratio in enumerate(ratios):
        if k == 0:
            hi, t = np.eye(3), torch.zeros(ty, tx, 2, device="cuda")
        else:
            hi = np.linalg.inv(_homography(rng, w, h))
            t = torch.randint(-shift, shift + 1, (ty, tx, 2), generator=g, device="cuda").float()
            far = torch.randint(-16, 17, (ty, tx, 2), generator=g, device="cuda").float()
            t = torch.where(_rand(g, ty, tx, 1) < movers, far, t)

        def back(x, y):
            d = hi[2, 0] * x + hi[2, 1] * y + hi[2, 2]
            zx = (hi[0, 0] * x + hi[0, 1] * y + hi[0, 2]) / d
            zy = (hi[1, 0] * x + hi[1, 1] * y + hi[1, 2]) / d
            q = t[(zy / TILE).floor().long().clamp(0, ty - 1),
                  (zx / TILE).floor().long().clamp(0, tx - 1)]
            return zx - q[..., 0] + m, zy - q[..., 1] + m

        yy, xx = torch.meshgrid(torch.arange(h, device="cuda").float(),
                                torch.arange(w, device="cuda").float(), indexing="ij")
        v = _sample(scene, *back(xx, yy)) * ratio
        v = v + (0.25 * v.clamp(min=0)).sqrt() * _randn(g, h, w) + 2.0 * _randn(g, h, w)
        planes = []
        if chroma is not None:
            yy, xx = torch.meshgrid(torch.arange(h // 2, device="cuda").float(),
                                    torch.arange(w // 2, device="cuda").float(), indexing="ij")
            at = back(2 * xx + 0.5, 2 * yy + 0.5)
            planes = [_u8(_sample(c, *at)) for c in chroma]
        if fmt == "nv12":
            uv = torch.stack(planes, -1).reshape(h // 2, w).contiguous()
            out.append(lnr.Frame(_u8(v), uv, None, float(ratio), True))
        else:
            out.append(lnr.Frame(_u8(v), *planes, exposure=float(ratio)) if planes
                       else lnr.Frame(_u8(v), exposure=float(ratio)))
    return out


def _equalised(y):
    """An image's 8-bit histogram equalisation (the guide and luma that stages take)."""
    cdf = torch.bincount(y.reshape(-1).int(), minlength=256).cumsum(0).double()
    low = cdf[cdf > 0][0]
    lut = ((cdf - low).clamp(min=0) * 255.0 / (cdf[-1] - low).clamp(min=1)).round()
    return lut.to(torch.uint8)[y.long()]


def _ctx():
    """The program's library context."""
    global _CTX
    if _CTX is None:
        _CTX = lnr.Context(torch.cuda.current_device())
    return _CTX


def _ratios(n):
    return tuple(4.0 ** k for k in range(n))


def _tiles(case, seed):
    """Network inputs (bf16 bits) as the pipeline makes them: 2x2 and 4x4 sums of a
    tile pair's pixels, and labels in the search range."""
    g = _gen(seed)
    n = case["tiles"]
    base = _smooth(g, 32 * 32, 32 * ((n + 31) // 32 + 1), 24.0, 90.0)
    k = torch.arange(n, device="cuda")
    lab = torch.randint(-14, 15, (n, 2), generator=g, device="cuda").int()
    ys = (k % 31) * 32
    xs = (k // 31) * 32
    r = torch.arange(16, device="cuda")
    chans = []
    for c in range(4):
        step, off = (2, 0) if c < 2 else (4, -16)
        yy = (ys.view(-1, 1, 1) + off + step * r.view(1, 16, 1)
              + (lab[:, 1].view(-1, 1, 1) if c & 1 else 0)).clamp(0, base.shape[0] - 1)
        xx = (xs.view(-1, 1, 1) + off + step * r.view(1, 1, 16)
              + (lab[:, 0].view(-1, 1, 1) if c & 1 else 0)).clamp(0, base.shape[1] - 1)
        chans.append(base[yy, xx] / 128.0 + 0.05 * _randn(g, n, 16, 16))
    x = torch.stack(chans, 1).clamp(-1, 1).to(torch.bfloat16).contiguous()
    return x, lab.contiguous()


def _weights(seed):
    """Network parameters: the shipped network for inference, He-normal ones to train."""
    if seed is None:
        return torch.from_numpy(proposal.load()[0]).cuda()
    g = _gen(seed)
    parts = []
    for co, ci in ((32, 4), (32, 32), (32, 32), (32, 32)):
        parts += [_randn(g, co * ci * 9) * math.sqrt(2.0 / (9 * ci)), 0.01 * _randn(g, co)]
    parts += [_randn(g, 3 * 512) * math.sqrt(1.0 / 512), 0.01 * _randn(g, 3)]
    return torch.cat(parts).float().contiguous()


def _batch_sizes(case):
    r = random.Random(case["sizes"])
    return [(2 * r.randint(320, max(320, case["max_width"] // 2)),
             2 * r.randint(240, max(240, case["max_height"] // 2))) for _ in range(case["pairs"])]


def _flow_inputs(case, seed):
    w, h = case["width"], case["height"]
    g = _gen(seed + 17)
    guide = _equalised(_frames(w, h, seed, (1.0, 4.0), "y8")[0].y)
    nx, ny = w // TILE, h // TILE
    step = torch.randint(-2, 3, (ny, nx, 2), generator=g, device="cuda") * 2
    ty, tx = torch.meshgrid(torch.arange(ny, device="cuda"), torch.arange(nx, device="cuda"),
                            indexing="ij")
    cxy = (torch.stack([tx, ty], -1) * TILE + TILE // 2 + step).reshape(-1, 2).int().contiguous()
    d = torch.stack([_smooth(g, ny, nx, 6.0, 9.0), _smooth(g, ny, nx, 6.0, 9.0)], -1)
    d = (d + 1.5 * _randn(g, ny, nx, 2)).round().clamp(-16, 16).reshape(-1, 2).int().contiguous()
    u = _rand(g, ny * nx)
    flags = torch.where(u < 0.25, torch.zeros_like(u), torch.where(u < 0.45, torch.full_like(u, 3),
                                                                    torch.full_like(u, 7)))
    return cxy, d, flags.to(torch.uint8).contiguous(), guide


def _warp_inputs(case, seed):
    w, h = case["width"], case["height"]
    g, rng = _gen(seed + 23), random.Random(seed + 23)
    src = _frames(w, h, seed, (1.0, 4.0), case["format"])[1]
    flow = torch.stack([_smooth(g, h, w, 40.0, 8.0), _smooth(g, h, w, 40.0, 8.0)]).contiguous()
    # normalised frame of the method: pixel = B (H C) with C, B of the image size
    hp = _homography(rng, w, h)
    c = np.array([[2.0, 0, -(w - 1)], [0, 2.0, -(h - 1)], [0, 0, w]])
    b = np.array([[w, 0, w - 1.0], [0, w, h - 1.0], [0, 0, 2.0]])
    hn = np.linalg.inv(b) @ hp @ np.linalg.inv(c)
    hn = torch.from_numpy(hn / hn[2, 2]).cuda().reshape(9).contiguous()
    return src, _equalised(src.y), hn, flow


def _merge_inputs(case, seed):
    """Frames and registrations as a program holds them before the merge."""
    w, h, n = case["width"], case["height"], case["frames"]
    frames = _frames(w, h, seed, _ratios(n), case["format"], shift=0, movers=0.05)
    g = _gen(seed + 31)
    regs = []
    yy, xx = torch.meshgrid(torch.arange(h, device="cuda").float(),
                            torch.arange(w, device="cuda").float(), indexing="ij")
    p = lnr.Params()
    for k in range(1, n):
        f = frames[k]
        at = (xx + _smooth(g, h, w, 60.0, 3.0), yy + _smooth(g, h, w, 60.0, 3.0))
        reg = lnr.Registration.alloc(w, h, f.fmt, p)
        ys = _sample(f.y.float(), *at)
        if f.u is None:
            reg.image[0] = ys / 255.0
        else:
            u, v = (f.u[:, 0::2], f.u[:, 1::2]) if f.nv12 else (f.u, f.v)
            us, vs = (_sample(q.float().contiguous(), at[0] / 2, at[1] / 2) - 128.0 for q in (u, v))
            reg.image[0] = (ys + 1.402 * vs) / 255.0
            reg.image[1] = (ys - 0.344136 * us - 0.714136 * vs) / 255.0
            reg.image[2] = (ys + 1.772 * us) / 255.0
        reg.yeq_warped.copy_(_sample(_equalised(f.y).float(), *at) / 255.0)
        reg.yeq_ref.copy_(_equalised(frames[0].y))
        regs.append(reg)
    return frames, regs


def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind, ctx=_ctx(), p=lnr.Params(radius0=case.get("radius", 16)))
    if kind == "pair":
        w, h = case["width"], case["height"]
        s["ref"], s["src"] = _frames(w, h, seed, (1.0, case["ratio"]), case["format"])
        if case["learned"]:
            s["ctx"] = lnr.Context(torch.cuda.current_device())
            lnr.proposal_set(s["ctx"], _weights(None))
            s["p"].learned, s["p"].conf_min = 1, proposal.load()[1]
        s["out"] = lnr.Registration.alloc(w, h, s["ref"].fmt, s["p"])
    elif kind == "stack":
        s["frames"] = _frames(case["width"], case["height"], seed, _ratios(case["frames"]),
                              case["format"], shift=12, movers=0.0, saturated=0.05)
    elif kind == "batch":
        pairs = [_frames(w, h, seed + 101 * i, (1.0, 2.0 + (5 * i) % 14), "i420", shift=16,
                         movers=0.0) for i, (w, h) in enumerate(_batch_sizes(case))]
        s["refs"], s["srcs"] = [q[0] for q in pairs], [q[1] for q in pairs]
        s["outs"] = [lnr.Registration.alloc(f.width, f.height, f.fmt, s["p"]) for f in s["refs"]]
    elif kind == "search":
        a, b = _frames(case["width"], case["height"], seed, (1.0, 8.0), "y8")
        s["ref"], s["warped"] = _equalised(a.y), _equalised(b.y)
    elif kind == "flow":
        s["cxy"], s["disp"], s["flags"], s["guide"] = _flow_inputs(case, seed)
    elif kind == "warp":
        s["src"], s["yeq"], s["H"], s["flow"] = _warp_inputs(case, seed)
    elif kind in ("merge", "irradiance"):
        s["frames"], s["regs"] = _merge_inputs(case, seed)
        f = s["frames"][0]
        s["out"] = torch.empty(1 if f.u is None else 3, f.height, f.width, device="cuda")
    else:
        s["ctx"] = lnr.Context(torch.cuda.current_device())
        s["x"], s["labels"] = _tiles(case, seed)
        s["params"] = _weights(None if kind == "forward" else seed + 3)
        lnr.proposal_set(s["ctx"], s["params"])
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------- run

_FIELDS = ("corner_xy", "disp", "ssd", "flags", "counts", "H", "yeq_ref", "yeq_src", "warped0",
           "flow", "ntilde", "image", "yeq_warped")


def _fields(reg):
    return {k: getattr(reg, k) for k in _FIELDS}


def run(s):
    kind, ctx, p = s["kind"], s["ctx"], s["p"]
    if kind == "pair":
        return _fields(lnr.register_pair(ctx, s["ref"], s["src"], p, out=s["out"]))
    if kind == "stack":
        regs, ref = lnr.register_stack(ctx, s["frames"], p)
        return dict(ref=ref, regs=[_fields(r) for r in regs])
    if kind == "batch":
        outs = lnr.register_batch(ctx, s["refs"], s["srcs"], p, outs=s["outs"])
        # every pair's flow and matches (a batch of 12 has more arrays than can be listed)
        return [dict(disp=r.disp, flags=r.flags, H=r.H, flow=r.flow, image=r.image) for r in outs]
    if kind == "search":
        return lnr.stage_search(ctx, s["ref"], s["warped"], p.radius0, p)
    if kind == "flow":
        return lnr.stage_flow(ctx, s["cxy"], s["disp"], s["flags"], s["guide"], p)
    if kind == "warp":
        return lnr.stage_backward_warp(ctx, s["src"], s["yeq"], s["H"], s["flow"])
    if kind == "merge":
        return lnr.merge(ctx, s["frames"], 0, s["regs"], p, out=s["out"])
    if kind == "irradiance":
        return lnr.merge_irradiance(ctx, s["frames"], 0, s["regs"], p, out=s["out"])
    if kind == "forward":
        return lnr.proposal_forward(ctx, s["x"])
    # the first step from these weights, so that every pass is the same step
    lnr.proposal_set(ctx, s["params"])
    loss, grad = lnr.proposal_train_step(ctx, s["x"], s["labels"], 3e-3, 1e-4, want_grad=True)
    return dict(loss=loss, grad=grad)


# ------------------------------------------------------------------ work

def _pair_work(w, h, fmt, radius, sources=1):
    n = w * h
    in_px = 1.0 if fmt == "y8" else 1.5
    ch = 1 if fmt == "y8" else 3
    # outputs per source: both equalised luma planes, the warped level, flow, N~, image, luma
    out_px = 3.0 + 8.0 + 4.0 + 4.0 * ch + 4.0
    # squared differences of 21 x 21 patches over the window of every level's tiles
    tiles, prod = n // (TILE * TILE), 0.0
    prod += tiles * 441.0 * (2 * radius + 1) ** 2
    prod += tiles / 3.0 * 441.0 * 21 ** 2
    # three propagation iterations of four directional sweeps over three maps
    return dict(bytes=n * (in_px * (1 + sources) + out_px * sources),
                flops=sources * (2.0 * prod + n * (3 * 4 * 3 * 3 + 60.0)))


def work(case):
    kind = case["kind"]
    if kind == "batch":
        each = [_pair_work(w, h, "i420", case["radius"]) for w, h in _batch_sizes(case)]
        return dict(bytes=sum(e["bytes"] for e in each), flops=sum(e["flops"] for e in each))
    if kind in ("forward", "train"):
        n, flop = case["tiles"], 2.0 * (256 * 36 * 32 + 2 * 64 * 288 * 32 + 16 * 288 * 32 + 1536)
        if kind == "forward":
            return dict(bytes=n * (2048 + 12) + 122e3, flops=n * flop)
        return dict(bytes=n * (2048 + 12) + 4 * 30467 * 7, flops=3 * n * flop)
    w, h = case["width"], case["height"]
    n = w * h
    in_px = {"y8": 1.0}.get(case.get("format"), 1.5)
    ch = 1 if case.get("format") == "y8" else 3
    if kind == "pair":
        return _pair_work(w, h, case["format"], case["radius"])
    if kind == "stack":
        return _pair_work(w, h, case["format"], case["radius"], case["frames"] - 1)
    if kind == "search":
        return dict(bytes=2.0 * n, flops=2.0 * (n // 1024) * 441 * (2 * case["radius"] + 1) ** 2)
    if kind == "flow":
        return dict(bytes=n * (1.0 + 12.0), flops=n * 3 * 4 * 3 * 3.0)
    if kind == "warp":
        return dict(bytes=n * (in_px + 1 + 8 + 4 * ch + 4), flops=n * 60.0)
    f = case["frames"]
    read = in_px + 1 + (f - 1) * (4.0 * ch + 4)
    ssim = (f - 1) * 2 * 11 * 4 * 2.0
    if kind == "irradiance":
        return dict(bytes=n * (read + 4 * ch), flops=n * (ssim + f * ch * 5))
    return dict(bytes=n * (read + 4 * ch), flops=n * (ssim + f * 40.0 + f * (ch + 1) * 10 * 4 / 3
                                                     + f * ch * 12 * 4 / 3))


# ----------------------------------------------------------------- exact

def _exact_flow(case, seed):
    """Recursive-filter domain transform in 64 bits: three iterations, rows then columns."""
    cxy, disp, flags, guide = _flow_inputs(case, seed)
    p = lnr.Params()
    h, w = guide.shape
    keep = (flags & 4) != 0
    m = torch.zeros(3, h, w, dtype=torch.float64, device="cuda")
    x, y = cxy[keep, 0].long(), cxy[keep, 1].long()
    m[0, y, x] = disp[keep, 0].double()
    m[1, y, x] = disp[keep, 1].double()
    m[2, y, x] = 1.0
    i = guide.double() / 255.0
    ratio = p.sigma_s / p.sigma_r
    dx = 1.0 + ratio * (i[:, 1:] - i[:, :-1]).abs()
    dy = 1.0 + ratio * (i[1:] - i[:-1]).abs()

    def sweep(m, c):  # along dimension 0 of m [n][3][lines], c [n - 1][1][lines], both ways
        for k in range(1, m.shape[0]):
            m[k] += c[k - 1] * (m[k - 1] - m[k])
        for k in range(m.shape[0] - 2, -1, -1):
            m[k] += c[k] * (m[k + 1] - m[k])
        return m

    n = p.dt_iters
    for k in range(1, n + 1):
        sig = p.sigma_s * math.sqrt(3.0) * 2.0 ** (n - k) / math.sqrt(4.0 ** n - 1.0)
        a = math.exp(-math.sqrt(2.0) / sig)
        t = sweep(m.permute(2, 0, 1).contiguous(), (a ** dx).t().contiguous()[:, None])
        t = sweep(t.permute(2, 1, 0).contiguous(), (a ** dy)[:, None])
        m = t.permute(1, 0, 2).contiguous()
    ok = m[2] > p.n_min
    flow = torch.where(ok, m[:2] / m[2], torch.zeros((), dtype=torch.float64, device="cuda"))
    return flow, m[2]


def _rgb(y, u, v):
    return torch.stack([(y + 1.402 * v) / 255.0, (y - 0.344136 * u - 0.714136 * v) / 255.0,
                        (y + 1.772 * u) / 255.0])


def _planes(f):
    """(Y, U, V) of a frame, chroma repeated to full size, in 64 bits."""
    if f.u is None:
        return f.y.double(), None, None
    u, v = (f.u[:, 0::2], f.u[:, 1::2]) if f.nv12 else (f.u, f.v)
    up = [q.double().repeat_interleave(2, 0).repeat_interleave(2, 1) for q in (u, v)]
    return f.y.double(), up[0], up[1]


def _exact_warp(case, seed):
    src, yeq, hn, flow = _warp_inputs(case, seed)
    w, h = case["width"], case["height"]
    hn = hn.cpu().numpy().reshape(3, 3)
    c = np.array([[2.0, 0, -(w - 1)], [0, 2.0, -(h - 1)], [0, 0, w]])
    b = np.array([[w, 0, w - 1.0], [0, w, h - 1.0], [0, 0, 2.0]])
    m = b @ (hn @ c)
    yy, xx = torch.meshgrid(torch.arange(h, device="cuda").double(),
                            torch.arange(w, device="cuda").double(), indexing="ij")
    x, y = xx + flow[0].double(), yy + flow[1].double()
    d = m[2, 0] * x + m[2, 1] * y + m[2, 2]
    sx = ((m[0, 0] * x + m[0, 1] * y + m[0, 2]) / d).clamp(-1, w)
    sy = ((m[1, 0] * x + m[1, 1] * y + m[1, 2]) / d).clamp(-1, h)
    x0, y0 = sx.floor(), sy.floor()
    ax, ay = sx - x0, sy - y0
    xa, xb = x0.long().clamp(0, w - 1), (x0.long() + 1).clamp(0, w - 1)
    ya, yb = y0.long().clamp(0, h - 1), (y0.long() + 1).clamp(0, h - 1)

    def bil(q):
        return ((1 - ay) * ((1 - ax) * q[ya, xa] + ax * q[ya, xb])
                + ay * ((1 - ax) * q[yb, xa] + ax * q[yb, xb]))

    y8, u, v = _planes(src)
    ys = bil(y8)
    img = (ys / 255.0)[None] if u is None else _rgb(ys, bil(u) - 128.0, bil(v) - 128.0)
    return img, bil(yeq.double()) / 255.0


def _clamped(x, r, dim):
    """x with r edge values repeated on both sides of a dimension."""
    n = x.shape[dim]
    i = torch.arange(-r, n + r, device=x.device).clamp(0, n - 1)
    return x.index_select(dim, i)


def _filter(x, taps):
    r = len(taps) // 2
    for dim in (-2, -1):
        q = _clamped(x, r, x.dim() + dim)
        n = x.shape[dim]
        x = sum(t * q.narrow(x.dim() + dim, k, n) for k, t in enumerate(taps))
    return x


def _exact_planes(case, seed):
    frames, regs = _merge_inputs(case, seed)
    y8, u, v = _planes(frames[0])
    imgs = [(y8 / 255.0)[None] if u is None else _rgb(y8, u - 128.0, v - 128.0)]
    imgs += [r.image.double() for r in regs]
    yeq = [regs[0].yeq_ref.double() / 255.0] + [r.yeq_warped.double() for r in regs]
    p = lnr.Params()
    taps = [math.exp(-j * j / (2.0 * p.ssim_sigma ** 2))
            for j in range(-p.ssim_radius, p.ssim_radius + 1)]
    taps = [t / sum(taps) for t in taps]
    ssim = [None]
    a = yeq[0]
    for b in yeq[1:]:
        ma, mb = _filter(a, taps), _filter(b, taps)
        va, vb = _filter(a * a, taps) - ma * ma, _filter(b * b, taps) - mb * mb
        cov = _filter(a * b, taps) - ma * mb
        ssim.append(((2 * ma * mb + p.ssim_c1) * (2 * cov + p.ssim_c2)
                     / ((ma * ma + mb * mb + p.ssim_c1) * (va + vb + p.ssim_c2))).clamp(min=0))
    return frames, imgs, ssim, p


def _exact_irradiance(case, seed):
    frames, imgs, ssim, _ = _exact_planes(case, seed)
    sw, se = torch.zeros_like(imgs[0]), torch.zeros_like(imgs[0])
    for f, v, q in zip(frames, imgs, ssim):
        wt = torch.minimum(v, 1.0 - v).clamp(min=0) * (1.0 if q is None else q)
        sw, se = sw + wt, se + wt * v / (f.exposure / frames[0].exposure)
    return torch.where(sw > 0, se / sw, imgs[0])


def _reduce(x):
    return _filter(x, [v / 16.0 for v in (1, 4, 6, 4, 1)])[..., ::2, ::2].contiguous()


def _expand(c, h, w):
    for dim, n in ((-1, w), (-2, h)):
        d = c.dim() + dim
        q = _clamped(c, 1, d)
        m = c.shape[d]
        lo, mid, hi = (q.narrow(d, k, m) for k in range(3))
        c = torch.stack([(lo + 6 * mid + hi) / 8.0, (mid + hi) / 2.0], d + 1)
        c = c.flatten(d, d + 1).narrow(d, 0, n)
    return c


def _exact_merge(case, seed):
    _, imgs, ssim, p = _exact_planes(case, seed)
    ws = []
    for v, q in zip(imgs, ssim):
        g = 0.299 * v[0] + 0.587 * v[1] + 0.114 * v[2] if v.shape[0] == 3 else v[0]
        e = _clamped(_clamped(g, 1, 0), 1, 1)
        wt = (e[:-2, 1:-1] + e[2:, 1:-1] + e[1:-1, :-2] + e[1:-1, 2:] - 4 * g).abs()
        if v.shape[0] == 3:
            wt = wt * ((v - v.mean(0)) ** 2).mean(0).sqrt()
        wt = wt * torch.exp(-((v - 0.5) ** 2).sum(0) / (2 * p.sigma_e ** 2))
        ws.append((wt if q is None else wt * q) + 1e-12)
    total = sum(ws)
    h, w = total.shape
    levels = 1
    while 8 << levels <= min(w, h):
        levels += 1
    acc = [None] * levels
    for v, wt in zip(imgs, ws):
        g, wt = v, (wt / total)[None]
        for l in range(levels):
            nxt = _reduce(g) if l + 1 < levels else None
            part = wt * (g if nxt is None else g - _expand(nxt, g.shape[-2], g.shape[-1]))
            acc[l] = part if acc[l] is None else acc[l] + part
            if nxt is not None:
                g, wt = nxt, _reduce(wt)
    r = acc[-1]
    for l in range(levels - 2, -1, -1):
        r = acc[l] + _expand(r, acc[l].shape[-2], acc[l].shape[-1])
    return r


def _bf(x):
    return x.float().to(torch.bfloat16).double()


_NET = ((32, 4, 1), (32, 32, 2), (32, 32, 1), (32, 32, 2))


def _network(params, x):
    """The network in 64 bits, rounded to bfloat16 where it is defined to be: weights and
    activations."""
    at, layers = 0, []
    p = params.double().cpu()
    for co, ci, s in _NET:
        n = co * ci * 9
        layers.append((_bf(p[at:at + n]).view(co, ci, 3, 3), p[at + n:at + n + co], s))
        at += n + co
    wh, bh = p[at:at + 1536].view(3, 512), p[at + 1536:]
    acts = [x.double().cpu()]
    for wt, b, s in layers:
        acts.append(_bf(F.conv2d(acts[-1], wt, b, stride=s, padding=1).clamp(min=0)))
    f = acts[-1].permute(0, 2, 3, 1).reshape(x.shape[0], 512)
    return layers, wh, acts, f, f @ wh.t() + bh


def _exact_forward(case, seed):
    x, _ = _tiles(case, seed)
    return _network(_weights(None), x)[-1]


def _exact_train(case, seed):
    x, labels = _tiles(case, seed)
    layers, wh, acts, f, o = _network(_weights(seed + 3), x)
    n = x.shape[0]
    lab = labels.double().cpu()
    e = 8.0 * o[:, :2] - lab
    z = o[:, 2]
    q = torch.sigmoid(4.0 * (2.5 - e.abs().max(1).values))
    hub = torch.where(e.abs() <= 1, 0.5 * e * e, e.abs() - 0.5).sum(1)
    loss = hub + z.clamp(min=0) - q * z + torch.log1p(torch.exp(-z.abs()))
    d = torch.cat([8.0 * e.clamp(-1, 1), (torch.sigmoid(z) - q)[:, None]], 1) / n
    gwh, gbh = d.t() @ f, d.sum(0)
    da = (d @ wh).view(n, 4, 4, 32).permute(0, 3, 1, 2)
    grads = []
    for k in range(3, -1, -1):
        wt, b, s = layers[k]
        dz = _bf(torch.where(acts[k + 1] > 0, da, torch.zeros_like(da)))
        gw = torch.nn.grad.conv2d_weight(acts[k], wt.shape, dz, stride=s, padding=1)
        grads.append((gw.reshape(-1), dz.sum((0, 2, 3))))
        if k:
            da = torch.nn.grad.conv2d_input(acts[k].shape, wt, dz, stride=s, padding=1)
    grad = torch.cat([t for gw, gb in reversed(grads) for t in (gw, gb)] + [gwh.reshape(-1), gbh])
    return dict(loss=loss, grad=grad)


def exact(case, seed):
    """The float outputs of the stages in 64 bits. A registration's matches are whole
    numbers, compared as they are; its flow and image follow from them through the
    propagation and the warp, whose values the flow and warp cases give."""
    kind = case["kind"]
    if kind == "flow":
        return _exact_flow(case, seed)
    if kind == "warp":
        return _exact_warp(case, seed)
    if kind == "merge":
        return _exact_merge(case, seed)
    if kind == "irradiance":
        return _exact_irradiance(case, seed)
    if kind == "forward":
        return _exact_forward(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    return None
