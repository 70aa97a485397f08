"""Edges of the kernels' work splits: the sizes where a split, a remainder or a
rule of a dispatch changes, each against the oracle or against another route
to the same values."""
import numpy as np
import pytest
import torch

import oracle
import synth
from test_gpu_proposal import _bf16_bits, _inputs, _offsets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lnr():
    import paper_1504_01441_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(lnr):
    return lnr.Context(0)


# gradient blocks of one sample, of two with a short last one, of four, the
# first size of the four-sample forward workgroup, more than 256 blocks' worth
@pytest.mark.parametrize("n", [1, 64, 65, 256, 257, 1030])
def test_training_step_at_block_edges(lnr, ctx, n):
    P = synth.proposal_params(11, head_scale=4.0)
    lnr.proposal_set(ctx, torch.from_numpy(P))
    x = _inputs(90 + n, n)
    lab = np.random.default_rng(n).integers(-10, 11, (n, 2)).astype(np.int32)
    xb, lb = _bf16_bits(x).cuda(), torch.from_numpy(lab).cuda()
    _, grad = lnr.proposal_train_step(ctx, xb, lb, 1e-3, 1e-4, want_grad=True)
    g = grad.cpu().numpy().astype(np.float64)
    _, g_o = oracle.cnn_loss_grad(P.astype(np.float64), x, lab, rnd=True)
    # bf16 activations that round the other way: 2 % of a tensor's norm (as in
    # test_gpu_proposal)
    for name, o, k in _offsets():
        nb = np.linalg.norm(g_o[o:o + k])
        assert np.linalg.norm(g[o:o + k] - g_o[o:o + k]) <= 2e-2 * nb + 1e-7, name
    # the step's packed weights are those of its parameters
    after = lnr.proposal_forward(ctx, xb)
    lnr.proposal_set(ctx, lnr.proposal_get(ctx))
    assert torch.equal(after, lnr.proposal_forward(ctx, xb))


def _homographies(w, h):
    """By kind: ordinary; a denominator that is 0 on a line through the frame;
    entries beyond (and far below) what the shared reciprocal takes; not finite."""
    a = np.array([[0.97, -0.05, 0.04], [0.06, 1.02, -0.03], [0.02, -0.03, 1.0]])
    cross = np.array([[1.0, 0.1, 0.0], [0.0, 1.0, 0.1], [1.0, 0.0, 0.0]])
    odd = a.copy()
    odd[0, 1] = np.nan
    return {"plain": a, "cross": cross, "huge": a * 1e150, "tiny": a * 1e-150, "nan": odd}


# the narrowest rows, whose two taps are not two bytes, rows that leave a
# thread 1, 2 and 3 of its 4 pixels, rows past one block
@pytest.mark.parametrize("w,h", [(1, 1), (1, 5), (2, 3), (3, 2), (5, 4), (1026, 3), (6, 40)])
def test_q8_warp_edges(lnr, ctx, w, h):
    img = np.random.default_rng(w * 7 + h).integers(0, 256, (h, w)).astype(np.uint8)
    for kind, H in _homographies(w, h).items():
        got = lnr.stage_warp_q8(ctx, torch.from_numpy(img).cuda(), torch.from_numpy(H.reshape(9)))
        want = oracle.warp_q8(img, oracle.pixel_homography(H, w, h))
        assert np.array_equal(got.cpu().numpy(), want), kind


# luma rows of one byte, chroma rows of one sample and two, one row per thread
# and (from 2 MP) four, with two rows left over
@pytest.mark.parametrize("fmt", ["y8", "i420", "nv12"])
@pytest.mark.parametrize("w,h", [(1, 3), (2, 2), (4, 6), (258, 6), (2048, 1030)])
def test_backward_warp_edges(lnr, ctx, w, h, fmt):
    if fmt != "y8" and w % 2:
        pytest.skip("4:2:0 frames are even")
    rng = np.random.default_rng(w + h)
    b = lambda *s: rng.integers(0, 256, s).astype(np.uint8)
    y, yeq, u, v = b(h, w), b(h, w), b(h // 2, w // 2), b(h // 2, w // 2)
    if fmt == "y8":
        u = v = None
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    f = (lnr.Frame.nv12_from_numpy(y, np.stack([u, v], 2).reshape(h // 2, w)) if fmt == "nv12"
         else lnr.Frame.from_numpy(y, u, v))
    flow = rng.uniform(-3, 3, (2, h, w)).astype(np.float32)
    flow[0, h // 2, w // 2] = 1e30  # far outside, on either side
    flow[1, 0, 0] = -1e38
    for kind, H in _homographies(w, h).items():
        img, yw = lnr.stage_backward_warp(ctx, f, t(yeq), torch.from_numpy(H.reshape(9)), t(flow))
        want, ywant = oracle.backward_warp(y, u, v, yeq, oracle.pixel_homography(H, w, h),
                                           flow[0].astype(np.float64), flow[1].astype(np.float64))
        # FP32 samples of values up to 2, the bound of the FP32 stages
        assert (np.abs(img.cpu().numpy() - want) <= 1e-4 * (np.abs(want) + 1.0)).all(), kind
        assert (np.abs(yw.cpu().numpy() - ywant) <= 1e-4 * (ywant + 1.0)).all(), kind


# one tile; a lane group of a wave and less; window energies summed by the
# candidates' threads and in runs; the last level with extra waves per tile and
# the first without
@pytest.mark.parametrize("nx,ny,R", [(1, 1, 0), (1, 1, 7), (2, 1, 1), (3, 2, 10), (5, 3, 8),
                                     (33, 31, 5), (32, 32, 5)])
@pytest.mark.parametrize("P", [1, 10])
def test_search_at_block_edges(lnr, ctx, nx, ny, R, P):
    rng = np.random.default_rng(nx * 100 + R)
    w, h = 32 * nx, 32 * ny
    base = np.kron(rng.integers(0, 256, (h // 8 + 4, w // 8 + 4)), np.ones((8, 8)))
    a = np.clip(base[3:3 + h, 5:5 + w] + rng.integers(-3, 4, (h, w)), 0, 255).astype(np.uint8)
    b = np.clip(base[1:1 + h, 2:2 + w] + rng.integers(-3, 4, (h, w)), 0, 255).astype(np.uint8)
    p, op = lnr.Params(patch_r=P), oracle.params(patch_r=P)
    t = lambda v: torch.from_numpy(v).cuda()
    cxy, disp, ssd, flags = (v.cpu().numpy() for v in lnr.stage_search(ctx, t(a), t(b), R, p))
    cx, cy, has = oracle.corners(a, op)
    dx, dy, want, valid = oracle.search(a, b, R, cx, cy, has, op)
    assert np.array_equal(flags & 1, has) and np.array_equal((flags & 2) > 0, valid > 0)
    v = valid > 0
    assert np.array_equal(disp[v, 0], dx[v]) and np.array_equal(disp[v, 1], dy[v])
    assert np.array_equal(ssd[v].view(np.uint32), want[v])


# windows past both sides, past one, ending with the row; rows aligned to a byte
@pytest.mark.parametrize("w,h", [(32, 32), (47, 33), (48, 40), (97, 64), (131, 97)])
def test_network_input_window_edges(lnr, ctx, w, h):
    rng = np.random.default_rng(w * h)
    ref, wrp = (rng.integers(0, 256, (h, w)).astype(np.uint8) for _ in range(2))
    x = lnr.proposal_inputs(ctx, torch.from_numpy(ref).cuda(), torch.from_numpy(wrp).cuda())
    want = oracle.cnn_tile_inputs(ref, wrp, range((w // 32) * (h // 32)))
    assert np.array_equal(x.view(torch.bfloat16).float().cpu().numpy(), want)


# the last one-sample workgroups and the first four-sample ones; rounds that
# leave 3, 2 and 1 of a workgroup's samples, a last round of few workgroups; an
# input aligned to its elements only. A sample's result does not depend on its
# place: the one-sample workgroups', which the oracle checks, give the same bits
@pytest.mark.parametrize("n", [256, 257, 1023, 1030, 2053])
@pytest.mark.parametrize("shift", [0, 1])
def test_forward_rounds(lnr, ctx, n, shift):
    P = synth.proposal_params(12, head_scale=4.0)
    lnr.proposal_set(ctx, torch.from_numpy(P))
    xb = _bf16_bits(_inputs(60 + n, n)).cuda()
    buf = torch.empty(xb.numel() + shift, dtype=xb.dtype, device="cuda")
    buf[shift:] = xb.reshape(-1)
    got = lnr.proposal_forward(ctx, buf[shift:].view(xb.shape))
    want = torch.cat([lnr.proposal_forward(ctx, xb[i:i + 200].contiguous())
                      for i in range(0, n, 200)])
    assert torch.equal(got, want)


# levels of staged tiles (more than 2^18 pixels) with ragged tiles and rows of 1,
# 2 and 3 pixels past the last four, of odd heights, and of one strip; the
# reduction's border strips and short row groups; stacks whose channels take
# more than one launch
@pytest.mark.parametrize("n,ch,w,h", [(2, 3, 513, 515), (2, 1, 4098, 67), (3, 3, 70, 4003),
                                      (2, 3, 1027, 512), (9, 3, 520, 509)])
def test_merge_at_tile_edges(lnr, ctx, n, ch, w, h):
    rng = np.random.default_rng(n * 1000 + w)
    step = np.ones((5, 5))
    plane = lambda: np.clip(np.kron(rng.uniform(0, 1, (h // 5 + 1, w // 5 + 1)), step)[:h, :w]
                            * 0.8 + rng.uniform(0, 0.2, (h, w)), 0, 1).astype(np.float32)
    imgs = [np.stack([plane() for _ in range(ch)]) for _ in range(n)]
    base = plane()
    yeqs = [np.clip(base + rng.uniform(-0.05, 0.05, (h, w)), 0, 1).astype(np.float32)
            for _ in range(n)]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    got = lnr.stage_merge(ctx, [t(i) for i in imgs], [t(y) for y in yeqs], 0, lnr.Params())
    want = oracle.merge([i.astype(np.float64) for i in imgs], [y.astype(np.float64) for y in yeqs],
                        0, oracle.params())
    # the bound of the FP32 stages
    assert (np.abs(got.cpu().numpy() - want) <= 1e-4 * (np.abs(want) + 1.0)).all()


# one word / two; the narrow and the wide hypothesis blocks; the last size of
# one fit block and the first of several; more iterations than blocks take at
# once, and counts that leave a group short; few matches with repeated draws
@pytest.mark.parametrize("nx,ny,iters,keep", [
    (5, 1, 1024, 1.0), (4, 2, 5, 0.6), (13, 5, 1023, 0.9), (16, 16, 37, 0.9), (257, 1, 1024, 0.9),
    (64, 32, 300, 0.8), (47, 45, 1024, 0.8), (70, 61, 3001, 0.7)])
def test_weeding_at_split_edges(lnr, ctx, nx, ny, iters, keep):
    rng = np.random.default_rng(nx * 100 + ny)
    p, op = lnr.Params(weed_iters=iters), oracle.params(weed_iters=iters)
    tile = 16 if nx > 190 else 32
    w, h = nx * tile, max(ny * tile, tile)
    gy, gx = np.mgrid[0:ny, 0:nx]
    cx = (gx * tile + tile // 2 + 2 * rng.integers(-2, 3, gx.shape)).ravel().astype(np.int32)
    cy = (gy * tile + tile // 2 + 2 * rng.integers(-2, 3, gx.shape)).ravel().astype(np.int32)
    dx = (np.rint(0.01 * (cx - w / 2) - 3) + rng.integers(-1, 2, cx.shape)).astype(np.int32)
    dy = (np.rint(0.02 * (cy - h / 2) + 2) + rng.integers(-1, 2, cx.shape)).astype(np.int32)
    far = rng.random(cx.shape) < 0.3
    dx[far], dy[far] = rng.integers(-16, 17, far.sum()), rng.integers(-16, 17, far.sum())
    valid = (rng.random(cx.shape) < keep).astype(np.uint8)
    M, n, bc, bi = oracle.weed(cx, cy, dx, dy, valid, w, h, 1, op)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    flags, H, counts = lnr.stage_weed_fit(
        ctx, t(np.stack([cx, cy], 1)), t(np.stack([dx, dy], 1)),
        t((valid * 3).astype(np.uint8)), w, h, 1, torch.eye(3, dtype=torch.float64).reshape(9), p)
    f, c = flags.cpu().numpy(), counts.cpu().numpy()
    assert np.array_equal((f & 4) > 0, M > 0)
    assert c[0] == valid.sum() and c[2] == bc and c[3] == bi
    sel = (f & 8) > 0
    assert c[1] == sel.sum() == (bc if bc > oracle.weed_delta(int(valid.sum()), op) else 0)
    want, _ = oracle.fit_level(cx, cy, dx, dy, sel.astype(np.uint8), w, h, np.eye(3))
    assert np.array_equal(H.cpu().numpy().reshape(3, 3), want)


# every default row and column shape at widths that are not whole 16-byte words
# or whole segments, and at lines shorter than one segment
@pytest.mark.parametrize("w,h", [(5, 40), (1021, 66), (2047, 40), (3070, 36), (4093, 33),
                                 (5002, 34), (40, 1023), (66, 2047), (35, 3071), (34, 4095),
                                 (33, 5001)])
def test_flow_at_line_edges(lnr, ctx, w, h):
    rng = np.random.default_rng(w + h)
    p, op = lnr.Params(), oracle.params()
    guide = np.clip(np.cumsum(rng.integers(-9, 10, (h, w)), 1) + 128, 0, 255).astype(np.uint8)
    nx, ny = w // 32, h // 32
    gy, gx = np.mgrid[0:ny, 0:nx]
    cx = (gx * 32 + 16 + rng.integers(-16, 16, gx.shape)).ravel().astype(np.int32)
    cy = (gy * 32 + 16 + rng.integers(-16, 16, gx.shape)).ravel().astype(np.int32)
    dx = rng.integers(-16, 17, cx.shape).astype(np.int32)
    dy = rng.integers(-16, 17, cx.shape).astype(np.int32)
    keep = (rng.random(cx.shape) < 0.7).astype(np.uint8)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    flow, nt = lnr.stage_flow(ctx, t(np.stack([cx, cy], 1).reshape(-1, 2)),
                              t(np.stack([dx, dy], 1).reshape(-1, 2)), t(keep * 7), t(guide), p)
    u, v, n = oracle.sparse_to_dense(cx, cy, dx, dy, keep, guide, op)
    mask = n > 2e-30
    for got, want in ((flow[0], u), (flow[1], v)):  # the FP32 stages' bound, 1e-4 relative
        err = np.abs(got.cpu().numpy().astype(np.float64) - want)
        assert (err <= 1e-4 * (np.abs(want) + 1.0))[mask].all()
    assert (np.abs(nt.cpu().numpy() - n) <= 1e-4 * (np.abs(n) + 1.0)).all()


# a negative n_min defines the flow everywhere as P~ / N~: infinite where the
# weight underflowed to 0 before the displacement did, undefined where both did
def test_flow_where_the_weight_underflows(lnr, ctx):
    w, h = 1600, 32
    flags = np.zeros(w // 32, np.uint8)
    flags[0] = 7
    cxy = np.stack([np.arange(w // 32) * 32 + 16, np.full(w // 32, 16)], 1).astype(np.int32)
    disp = np.tile(np.array([16, -16], np.int32), (w // 32, 1))
    t = lambda a: torch.from_numpy(a).cuda()
    flow, nt = (v.cpu().numpy() for v in lnr.stage_flow(
        ctx, t(cxy), t(disp), t(flags), torch.zeros(h, w, dtype=torch.uint8, device="cuda"),
        lnr.Params(sigma_s=8.0, n_min=-1.0)))
    assert (np.abs(flow[0][nt > 1e-30] - 16) < 1e-3).all()
    zero = nt == 0
    inf = np.isposinf(flow[0])
    # 16 N~ leaves the floats four powers of two after N~ does, at 0.82 per pixel
    assert inf[zero].sum() >= h and not inf[~zero].any()
    assert np.array_equal(inf, np.isneginf(flow[1]))
    assert np.isnan(flow[:, zero & ~inf]).all()


def _weeding_case(nx, ny, tile, keep, seed):
    """Matches of one level: a smooth motion with rounding, a third of them
    random, `keep` of the tiles valid: (w, h, cx, cy, dx, dy, valid)."""
    rng = np.random.default_rng(seed)
    w, h = nx * tile, ny * tile
    gy, gx = np.mgrid[0:ny, 0:nx]
    cx = (gx * tile + tile // 2 + rng.integers(-2, 3, gx.shape)).ravel().astype(np.int32)
    cy = (gy * tile + tile // 2 + rng.integers(-2, 3, gx.shape)).ravel().astype(np.int32)
    dx = (np.rint(0.002 * (cx - w / 2) - 3) + rng.integers(-1, 2, cx.shape)).astype(np.int32)
    dy = (np.rint(0.003 * (cy - h / 2) + 2) + rng.integers(-1, 2, cx.shape)).astype(np.int32)
    far = rng.random(cx.shape) < 0.3
    dx[far], dy[far] = rng.integers(-16, 17, far.sum()), rng.integers(-16, 17, far.sum())
    return w, h, cx, cy, dx, dy, (rng.random(cx.shape) < keep).astype(np.uint8)


def _weeding_parity(lnr, ctx, case, iters):
    w, h, cx, cy, dx, dy, valid = case
    p, op = lnr.Params(weed_iters=iters), oracle.params(weed_iters=iters)
    M, n, bc, bi = oracle.weed(cx, cy, dx, dy, valid, w, h, 1, op)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    flags, H, counts = lnr.stage_weed_fit(
        ctx, t(np.stack([cx, cy], 1)), t(np.stack([dx, dy], 1)),
        t((valid * 3).astype(np.uint8)), w, h, 1, torch.eye(3, dtype=torch.float64).reshape(9), p)
    f, c = flags.cpu().numpy(), counts.cpu().numpy()
    assert np.array_equal((f & 4) > 0, M > 0)
    assert c[0] == valid.sum() and c[2] == bc and c[3] == bi
    sel = (f & 8) > 0
    assert c[1] == sel.sum() == (bc if bc > oracle.weed_delta(int(valid.sum()), op) else 0)
    want, _ = oracle.fit_level(cx, cy, dx, dy, sel.astype(np.uint8), w, h, np.eye(3))
    assert np.array_equal(H.cpu().numpy().reshape(3, 3), want)


# the largest level: 2304 tile words
@pytest.mark.parametrize("iters", [37, 1100])
def test_weeding_of_the_largest_level(lnr, ctx, iters):
    _weeding_parity(lnr, ctx, _weeding_case(384, 384, 16, 0.8, iters), iters)


# batches of pairs whose level 0 has the most tile words that eight hypotheses
# per block can hold (1938, from four pairs on) and more: the single calls'
# results, which take four per block
@pytest.mark.parametrize("n,H", [(2, 5184), (4, 5168), (4, 5184)])
def test_batch_with_a_level_of_many_tiles(lnr, ctx, n, H):
    rng = np.random.default_rng(n)
    p = lnr.Params(tile=16, patch_r=3, quad_r=3, corner_step=1, radius0=2, radius_coarse=2,
                   weed_iters=50, dt_iters=1)
    frames = []
    for w, h in [(6144, H)] + [(320, 200)] * (n - 1):
        y = rng.integers(0, 256, (h, w), dtype=np.uint8)
        frames.append((lnr.Frame.from_numpy(y), lnr.Frame.from_numpy(np.roll(y, (1, -1), (0, 1)))))
    refs, srcs = [f[0] for f in frames], [f[1] for f in frames]
    outs = lnr.register_batch(ctx, refs, srcs, p)
    for r, s, got in zip(refs, srcs, outs):
        want = lnr.register_pair(ctx, r, s, p)
        torch.cuda.synchronize()
        for k in ("corner_xy", "disp", "ssd", "flags", "counts", "H", "flow", "image"):
            a, b = getattr(got, k), getattr(want, k)
            assert torch.equal(a, b), k


# the fixed scratch filled to its last byte: one weeding iteration, whose
# buffers are the smallest part of a plan, in a frame that leaves no room
def test_noalloc_at_the_scratch_limit(lnr, ctx):
    w, h = 1021, 5912
    p = lnr.Params(tile=16, patch_r=3, quad_r=3, corner_step=1, radius0=2, radius_coarse=2,
                   weed_iters=1, dt_iters=3)
    rng = np.random.default_rng(w)
    y = np.kron(rng.integers(0, 256, (h // 4, w // 4 + 1)), np.ones((4, 4)))[:, :w].astype(np.uint8)
    ref, src = lnr.Frame.from_numpy(y), lnr.Frame.from_numpy(np.roll(y, (1, -1), (0, 1)))
    got = lnr.Registration.alloc(w, h, lnr.LNR_Y8, p)
    lnr.register_pair_noalloc(ctx, ref, src, p, out=got)
    want = lnr.register_pair(ctx, ref, src, p)
    torch.cuda.synchronize()
    for k in ("corner_xy", "disp", "ssd", "flags", "H", "flow", "image"):
        assert torch.equal(getattr(got, k), getattr(want, k)), k


def _flow_case(w, h, seed):
    """Corners of every tile, displacements, the kept ones, and a guide."""
    rng = np.random.default_rng(seed)
    guide = np.clip(np.cumsum(rng.integers(-9, 10, (h, w)), 1) + 128, 0, 255).astype(np.uint8)
    gy, gx = np.mgrid[0:h // 32, 0:w // 32]
    cx = (gx * 32 + 16 + rng.integers(-16, 16, gx.shape)).ravel().astype(np.int32)
    cy = (gy * 32 + 16 + rng.integers(-16, 16, gx.shape)).ravel().astype(np.int32)
    dx, dy = (rng.integers(-16, 17, cx.shape).astype(np.int32) for _ in range(2))
    return cx, cy, dx, dy, (rng.random(cx.shape) < 0.7).astype(np.uint8), guide


# the default column shapes from the first to the last height that takes them:
# segments of 12, 20 and 24 rows (test_flow_at_line_edges has the others)
@pytest.mark.parametrize("w,h", [(40, 1025), (37, 1536), (33, 2049), (34, 2560), (35, 2561),
                                 (33, 4097), (36, 5121), (33, 6144)])
def test_flow_default_column_shapes(lnr, ctx, w, h):
    p, op = lnr.Params(), oracle.params()
    cx, cy, dx, dy, keep, guide = _flow_case(w, h, w + h)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    flow, nt = lnr.stage_flow(ctx, t(np.stack([cx, cy], 1)), t(np.stack([dx, dy], 1)),
                              t(keep * 7), t(guide), p)
    u, v, n = oracle.sparse_to_dense(cx, cy, dx, dy, keep, guide, op)
    mask = n > 2e-30
    for got, want in ((flow[0], u), (flow[1], v)):  # the FP32 stages' bound, 1e-4 relative
        err = np.abs(got.cpu().numpy().astype(np.float64) - want)
        assert (err <= 1e-4 * (np.abs(want) + 1.0))[mask].all()
    assert (np.abs(nt.cpu().numpy() - n) <= 1e-4 * (np.abs(n) + 1.0)).all()


# the column shapes that only the tuner takes, at the first and last heights
# that have each: 4 rows by 128 segments in blocks of four columns,
# and 4, 8 and 12 rows by 256 segments
@pytest.mark.parametrize("w,h,l,nseg", [
    (37, 32, 4, 128), (40, 511, 4, 128), (33, 512, 4, 128), (36, 130, 4, 256), (35, 1024, 4, 256),
    (38, 1025, 8, 256), (33, 2048, 8, 256), (40, 2049, 12, 256), (37, 3000, 12, 256),
    (34, 3072, 12, 256)])
def test_flow_column_shapes_of_the_tuner(lnr, w, h, l, nseg):
    c = lnr.Context(0)
    p, op = lnr.Params(), oracle.params()
    lnr.set_flow_shape(c, w, h, (4, 256, l, 4, nseg))
    cx, cy, dx, dy, keep, guide = _flow_case(w, h, w + h)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    flow, nt = lnr.stage_flow(c, t(np.stack([cx, cy], 1)), t(np.stack([dx, dy], 1)),
                              t(keep * 7), t(guide), p)
    u, v, n = oracle.sparse_to_dense(cx, cy, dx, dy, keep, guide, op)
    mask = n > 2e-30
    for got, want in ((flow[0], u), (flow[1], v)):  # the FP32 stages' bound, 1e-4 relative
        err = np.abs(got.cpu().numpy().astype(np.float64) - want)
        assert (err <= 1e-4 * (np.abs(want) + 1.0))[mask].all()
    assert (np.abs(nt.cpu().numpy() - n) <= 1e-4 * (np.abs(n) + 1.0)).all()
    with pytest.raises(lnr.LnrError):  # not the fewest rows, and not listed
        lnr.set_flow_shape(c, w, h, (4, 256, l + 4, 4, 256))
    c.close()


# a pinned shape's rows per segment are the rows that run, whatever the height
# needs: where a segment ends shows in the last bits of the flow, so that other
# rows give other bits (within the bound), and the same pin gives the same
def test_pinned_flow_shapes_are_the_ones_that_run(lnr):
    c = lnr.Context(0)
    w, h = 640, 480
    rng = np.random.default_rng(3)
    y = np.kron(rng.integers(0, 256, (h // 8, w // 8)), np.ones((8, 8)))
    y = np.clip(y + rng.integers(-3, 4, (h, w)), 0, 255).astype(np.uint8)
    ref, src = lnr.Frame.from_numpy(y), lnr.Frame.from_numpy(np.roll(y, (2, -3), (0, 1)))
    p = lnr.Params(radius0=8)

    def run(shape):
        lnr.set_flow_shape(c, w, h, shape)
        return lnr.register_pair(c, ref, src, p).ntilde.cpu().numpy()

    got = {rows: run((4, 256, rows, 4, 128)) for rows in (8, 16, 24)}
    for a, b in ((8, 16), (8, 24), (16, 24)):
        assert not np.array_equal(got[a], got[b])
        assert (np.abs(got[a] - got[b]) <= 1e-4 * (np.abs(got[a]) + 1.0)).all()
    assert np.array_equal(got[16], run((4, 256, 16, 4, 128)))
    # what the tuner reports can be pinned, also where the default is not listed
    for size in ((w, h), (700, 1080)):
        shape = lnr.autotune_flow(c, *size, p)
        assert shape[0] * shape[1] >= size[0] and shape[2] * shape[4] >= size[1]
        lnr.set_flow_shape(c, *size, shape)
    with pytest.raises(lnr.LnrError):
        lnr.set_flow_shape(c, w, h, (4, 256, 12, 4, 128))  # the default of another height
    c.close()


# iterations beyond one group per block: the last and first counts that one
# wave, two, a part of one and all waves of a block solve, and a second turn of
# the blocks; narrow blocks (up to 256 tiles), then wide ones
@pytest.mark.parametrize("nx,ny,iters", [
    (12, 9, 2048), (12, 9, 2049), (12, 9, 8192), (12, 9, 8193), (5, 3, 20000),
    (20, 15, 1025), (20, 15, 2049), (20, 15, 16384), (20, 15, 16389), (70, 61, 16389)])
def test_weeding_of_many_iterations(lnr, ctx, nx, ny, iters):
    _weeding_parity(lnr, ctx, _weeding_case(nx, ny, 32, 0.8, iters + nx), iters)


# few iterations over many tiles, tested in chunks of tiles: the first level
# that takes chunks and the last that does not, a single iteration, groups left
# short, the most hypotheses of the narrow and of the wide sums of the chunks'
# counts and the first past them, chunks of one and of several turns; so few
# valid matches that no hypothesis is usable
@pytest.mark.parametrize("nx,ny,iters,keep", [
    (64, 48, 17, 0.8), (61, 51, 17, 0.8), (61, 51, 1, 0.8), (61, 51, 256, 0.8),
    (61, 51, 257, 0.8), (129, 65, 300, 0.8), (129, 65, 512, 0.8), (129, 65, 513, 0.8),
    (250, 186, 5, 0.8), (250, 186, 128, 0.8), (250, 186, 129, 0.5), (70, 61, 40, 0.0005)])
def test_weeding_of_few_iterations(lnr, ctx, nx, ny, iters, keep):
    _weeding_parity(lnr, ctx, _weeding_case(nx, ny, 16, keep, iters + nx), iters)


# a batch's levels in chunks, with pairs that have one and a few of them
@pytest.mark.parametrize("iters", [3, 64, 400])
@pytest.mark.parametrize("n", [1, 3, 5])
def test_batch_of_few_iterations(lnr, ctx, n, iters):
    rng = np.random.default_rng(n)
    p = lnr.Params(tile=16, patch_r=3, quad_r=3, corner_step=1, radius0=2, radius_coarse=2,
                   weed_iters=iters, dt_iters=1)
    frames = []
    for w, h in [(2592, 1944), (17, 16), (700, 500), (320, 200), (1000, 1300)][:n]:
        y = np.kron(rng.integers(0, 256, (h // 4 + 1, w // 4 + 1)), np.ones((4, 4)))
        y = y[:h, :w].astype(np.uint8)
        frames.append((lnr.Frame.from_numpy(y), lnr.Frame.from_numpy(np.roll(y, (1, -1), (0, 1)))))
    refs, srcs = [f[0] for f in frames], [f[1] for f in frames]
    for graph in (False, True):
        outs = lnr.register_batch(ctx, refs, srcs, p, graph=graph)
        for r, s, got in zip(refs, srcs, outs):
            want = lnr.register_pair(ctx, r, s, p)
            torch.cuda.synchronize()
            for k in ("corner_xy", "disp", "ssd", "flags", "counts", "H", "flow", "image"):
                assert torch.equal(getattr(got, k), getattr(want, k)), k


# the automatic search shapes on both sides of every line between them: the
# matrix cores at radius 11 and below (from 2048 tiles), their patch-row groups
# by the number of tiles, the patches and quadrants that go to the lanes, and
# radius 32 on few tiles
@pytest.mark.parametrize("tile,nx,ny,R,P,r", [
    (32, 1, 1, 11, 1, 10), (32, 1, 1, 11, 10, 10), (32, 3, 1, 16, 1, 10), (32, 2, 1, 16, 10, 10),
    (32, 1, 2, 24, 1, 10), (32, 1, 3, 24, 10, 10), (32, 1, 1, 32, 10, 10), (32, 3, 1, 32, 4, 10),
    (32, 23, 89, 8, 10, 10), (32, 32, 64, 8, 10, 10), (32, 23, 89, 10, 7, 3),
    (32, 32, 64, 10, 7, 3), (16, 24, 20, 11, 3, 3), (16, 13, 37, 11, 3, 3), (16, 25, 32, 11, 5, 3),
    (16, 9, 89, 11, 5, 3), (16, 20, 16, 16, 2, 3), (16, 3, 107, 16, 2, 3), (16, 64, 65, 10, 3, 3),
    (16, 49, 85, 10, 3, 3), (16, 49, 85, 10, 5, 5), (32, 64, 81, 8, 5, 5), (32, 64, 81, 8, 5, 6),
    (16, 15, 17, 32, 3, 3), (16, 16, 16, 32, 3, 3), (16, 15, 17, 32, 1, 2), (16, 15, 17, 32, 4, 3)])
def test_automatic_search_shapes(lnr, ctx, tile, nx, ny, R, P, r):
    rng = np.random.default_rng(nx * 100 + R)
    w, h = tile * nx, tile * ny
    base = np.kron(rng.integers(0, 256, (h // 4 + 4, w // 4 + 4)), np.ones((4, 4)))
    a = np.clip(base[3:3 + h, 5:5 + w] + rng.integers(-3, 4, (h, w)), 0, 255).astype(np.uint8)
    b = np.clip(base[1:1 + h, 2:2 + w] + rng.integers(-3, 4, (h, w)), 0, 255).astype(np.uint8)
    kw = dict(tile=tile, patch_r=P, quad_r=r, corner_step=1, min_level_dim=64)
    p, op = lnr.Params(**kw), oracle.params(**kw)
    t = lambda v: torch.from_numpy(v).cuda()
    cxy, disp, ssd, flags = (v.cpu().numpy() for v in lnr.stage_search(ctx, t(a), t(b), R, p))
    cx, cy, has = oracle.corners(a, op)
    dx, dy, want, valid = oracle.search(a, b, R, cx, cy, has, op)
    assert np.array_equal(flags & 1, has) and np.array_equal((flags & 2) > 0, valid > 0)
    v = valid > 0
    assert v.any() or nx * ny < 4
    assert np.array_equal(disp[v, 0], dx[v]) and np.array_equal(disp[v, 1], dy[v])
    assert np.array_equal(ssd[v].view(np.uint32), want[v])
