"""The blend, projection and binning kernels at the edges of their rounds, list
cuts, quarter masks and rectangle queues, against the FP64 oracle (tolerances and guard band of the render
parity tests: images 1e-4, gradients 1e-3)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import (GRAD_TOL, IMG_TOL, check_binning_self_consistent, guard_report, log, oracle_opts, rel_err,
                            to_np, upstream)

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2505_22335_amd as P
    from paper_2505_22335_amd import _lib as L


def _check(sc, cam, nf, label, max_frac, grads=("mean", "scale", "rot", "opacity", "rgb")):
    ref = oracle.render_scene(sc, cam, oracle_opts(nf), with_margins=True)
    keep, rep = guard_report(ref["margins"], tie_ulps=0)
    log("case", label, rep)
    assert rep["frac"] <= max_frac, rep
    G = upstream(5, cam.height, cam.width, nf)
    G = {k: v * keep for k, v in G.items()}
    _, gr = oracle.render_scene(sc, cam, oracle_opts(nf), grad_out=G, pose_grad=True)
    g = P.gaussians_to_device(sc.arrays())
    rc = P.RenderContext([cam], sc.n, n_feat=nf)
    rc.fit(g)
    out = rc.forward(g)
    dg, dpose = rc.backward(g, {k: torch.as_tensor(v[None].astype(np.float32)).cuda() for k, v in G.items()})
    torch.cuda.synchronize()
    for k in ("rgb", "depth", "alpha") + (("feat",) if nf else ()):
        e = rel_err(to_np(out[k][0]), ref[k], keep)
        assert e <= IMG_TOL, (label, k, e)
    for k in grads + (("feat",) if nf else ()):
        e = rel_err(to_np(dg[k][0]), gr["gauss"][k])
        assert e <= GRAD_TOL, (label, k, e)
    e = rel_err(to_np(dpose[0]), gr["pose"])
    assert e <= GRAD_TOL, (label, "pose", e)


@pytest.mark.parametrize("nf", [0, 16])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 31, 32, 33, 128, 129, 255, 256, 257, 513, 1100])
def test_one_tile_list_lengths(n, nf):
    """n wide faint Gaussians over one 16x16 tile: batches of 8, rounds of 32
    and 256 entries, and lists cut from 129 entries on."""
    rng = np.random.default_rng(n)
    z = rng.uniform(2.0, 4.0, n)
    q = rng.normal(size=(4, n))
    sc = synth.PlainScene(
        mean=np.stack([rng.uniform(-0.2, 0.2, n), rng.uniform(-0.2, 0.2, n), z]).astype(np.float32),
        scale=rng.uniform(1.5, 4.0, (3, n)).astype(np.float32), rot=(q / np.linalg.norm(q, axis=0)).astype(np.float32),
        opacity=rng.uniform(0.006, 0.02, n).astype(np.float32), rgb=rng.uniform(0, 1, (3, n)).astype(np.float32),
        feat=rng.normal(size=(nf, n)).astype(np.float32) if nf else None)
    cam = synth.Camera(16, 16, 20.0, 20.0, 7.5, 7.5, np.eye(3, 4, dtype=np.float32))
    _check(sc, cam, nf, "one tile n=%d nf=%d" % (n, nf), 0.15)


def _box_and_power(geom, W, H):
    """Half extents of each Gaussian's reach box (slot 7, two half floats) and
    the kernels' float32 power at every pixel, (n, H, W): products and sums in
    the kernels' order, fused steps rounded once."""
    f = np.float32
    box = geom[:, 7].copy().view(np.uint32)
    hx = (box & 0xFFFF).astype(np.uint16).view(np.float16).astype(f)
    hy = (box >> 16).astype(np.uint16).view(np.float16).astype(f)
    u, v, A, B, C = (geom[:, i][:, None, None] for i in range(5))
    dx = (u - np.arange(W, dtype=f)[None, None, :]).astype(f)
    dy = (v - np.arange(H, dtype=f)[None, :, None]).astype(f)
    fma = lambda a, b, c: (a.astype(np.float64) * b + c).astype(f)  # noqa: E731
    with np.errstate(over="ignore", invalid="ignore"):
        q = fma((C * dy).astype(f), dy, ((A * dx).astype(f) * dx).astype(f))
        return hx, hy, dx, dy, fma(np.float32(-0.5) * np.ones_like(q), q, -((B * dx).astype(f) * dy).astype(f))


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("seed", [0, 1])
def test_reach_box_holds_every_used_pixel(seed, mode):
    """Needles of axis ratio up to 1e4, blobs wider than the image by orders
    of magnitude, specks below a pixel and opacities at both ends: every pixel
    that passes the kernels' alpha test lies inside the box the quarter masks
    are formed from (the masks leave no used pixel out)."""
    rng = np.random.default_rng(40 + seed)
    n = 120
    z = rng.uniform(1.5, 4.0, n)
    scale = np.exp(rng.uniform(np.log(1e-3), np.log(0.3), (3, n)))
    scale[0, :30] = rng.uniform(0.5, 10.0, 30)   # needles
    scale[1:, :30] = 10.0 ** rng.uniform(-3.0, -1.5, (2, 30))
    scale[:, 30:36] = 10.0 ** rng.uniform(1.0, 3.0, (3, 6))  # blobs
    o = rng.uniform(0.02, 0.9, n)
    o[30:36] = 0.01
    o[100:110] = 0.0045
    q = rng.normal(size=(4, n))
    sc = synth.PlainScene(
        mean=np.stack([rng.uniform(-0.8, 0.8, n) * z / 2, rng.uniform(-0.8, 0.8, n) * z / 2, z]).astype(np.float32),
        scale=scale.astype(np.float32), rot=q.astype(np.float32), opacity=o.astype(np.float32),
        rgb=rng.uniform(0, 1, (3, n)).astype(np.float32))
    W, H = 75, 53
    cam = synth.Camera(W, H, 60.0, 60.0, 37.0, 26.0, np.eye(3, 4, dtype=np.float32))
    g = P.gaussians_to_device(sc.arrays())
    rc = P.RenderContext([cam], n, n_feat=0, extent_mode=mode)
    rc.fit(g)
    rc.forward(g)
    seen = rc.array(L.CTX_NTILES, torch.int32).cpu().numpy() > 0
    geom = rc.array(L.CTX_GEOM, torch.float32, width=8).cpu().numpy()[seen]
    hx, hy, dx, dy, power = _box_and_power(geom, W, H)
    used = (power <= 0) & (power >= geom[:, 6][:, None, None])
    outside = (np.abs(dx) > hx[:, None, None]) | (np.abs(dy) > hy[:, None, None])
    log("case reach box", seed, mode, "used", int(used.sum()), "outside", int((used & outside).sum()))
    assert used.sum() > 1000
    assert not np.any(used & outside)


def _quarter_stops_scene(n, nf):
    """n specks over one 16x16 tile; the upper left quarter is closed by opaque
    ones 40 entries into the sixth of sixteen equal list segments."""
    rng = np.random.default_rng(n + nf)
    z = np.linspace(2.0, 4.0, n)
    u, v = rng.uniform(-0.5, 15.5, n), rng.uniform(-0.5, 15.5, n)
    sig, o = rng.uniform(1.0, 2.0, n), rng.uniform(0.006, 0.03, n)
    seg = -(-(-(-n // 16)) // 32) * 32
    a = 5 * seg + 40
    k = np.arange(100)
    u[a:a + 100], v[a:a + 100] = 2.0 + 3.0 * (k & 1), 2.0 + 3.0 * ((k >> 1) & 1)
    sig[a:a + 100], o[a:a + 100] = 2.0, 0.9
    f = 20.0
    sc = synth.PlainScene(
        mean=np.stack([(u - 7.5) * z / f, (v - 7.5) * z / f, z]).astype(np.float32),
        scale=np.broadcast_to(sig * z / f, (3, n)).astype(np.float32),
        rot=np.broadcast_to(np.array([1.0, 0.0, 0.0, 0.0])[:, None], (4, n)).astype(np.float32),
        opacity=o.astype(np.float32), rgb=rng.uniform(0, 1, (3, n)).astype(np.float32),
        feat=rng.normal(size=(nf, n)).astype(np.float32) if nf else None)
    return sc, synth.Camera(16, 16, f, f, 7.5, 7.5, np.eye(3, 4, dtype=np.float32))


@pytest.mark.parametrize("nf", [0, 16])
@pytest.mark.parametrize("n", [4300, 6000, 8100])
def test_quarter_stops_inside_a_long_segment(n, nf):
    """List segments of more than one round of 256 entries (288, 384, 512), one
    quarter of the tile closed in a segment's first round while the others go on
    past its end: that quarter recorded no state at the segment's end, and the
    walk of the segment starts from its pixels' final state there."""
    sc, cam = _quarter_stops_scene(n, nf)
    # the specks are round: no gradient reaches their rotation
    _check(sc, cam, nf, "quarter stops n=%d nf=%d" % (n, nf), 0.15, ("mean", "scale", "opacity", "rgb"))


@pytest.mark.parametrize("nf", [0, 16])
@pytest.mark.parametrize("n", [3, 33, 300])
def test_gradients_over_many_tiles(n, nf):
    """Strips over up to 18 x 2 tiles of a 288x24 image, between specks: the
    projection's backward sums up to 16 tiles in the Gaussian's thread and more
    in a wave."""
    rng = np.random.default_rng(n + nf)
    z = rng.uniform(2.0, 4.0, n)
    f = 100.0
    u, v = rng.uniform(110.0, 178.0, n), rng.uniform(2.0, 22.0, n)
    wide = np.arange(n) % 3 != 2
    sx, sy = np.where(wide, rng.uniform(35.0, 60.0, n), 1.5), rng.uniform(0.8, 2.5, n)
    q = np.stack([np.ones(n), 0.01 * rng.normal(size=n), 0.01 * rng.normal(size=n), 0.01 * rng.normal(size=n)])
    sc = synth.PlainScene(
        mean=np.stack([(u - 143.5) * z / f, (v - 11.5) * z / f, z]).astype(np.float32),
        scale=np.stack([sx * z / f, sy * z / f, sy * z / f]).astype(np.float32), rot=q.astype(np.float32),
        opacity=rng.uniform(0.05, 0.6, n).astype(np.float32), rgb=rng.uniform(0, 1, (3, n)).astype(np.float32),
        feat=rng.normal(size=(nf, n)).astype(np.float32) if nf else None)
    cam = synth.Camera(288, 24, f, f, 143.5, 11.5, np.eye(3, 4, dtype=np.float32))
    rc = P.RenderContext([cam], n, n_feat=nf)
    g = P.gaussians_to_device(sc.arrays())
    rc.fit(g)
    rc.forward(g)
    tiles = rc.array(L.CTX_NTILES, torch.int32).cpu().numpy()
    log("case many tiles", n, nf, "largest", int(tiles.max()), "16:", int((tiles == 16).sum()), "17:", int((tiles == 17).sum()))
    assert tiles.max() > 16 and (n < 300 or ((tiles == 16).any() and (tiles == 17).any()))
    _check(sc, cam, nf, "many tiles n=%d nf=%d" % (n, nf), 0.15)


@pytest.mark.parametrize("n", [5, 256, 700])
@pytest.mark.parametrize("W,H", [(640, 480), (1024, 1024), (1040, 1024)])
def test_binning_of_wide_rectangles(W, H, n):
    """Rectangles of one tile to several hundred in views of 1200, 4096 (the
    LDS grid's limit) and 4160 tiles: small ones by their thread, larger ones
    by a wave, over the grid or the global counters. Lists, ranges and order
    equal their integer re-derivation."""
    rng = np.random.default_rng(W + n)
    z = rng.uniform(2.0, 4.0, n)
    f = 500.0
    px = np.exp(rng.uniform(np.log(1.0), np.log(70.0), (2, n)))  # standard deviations in pixels
    q = rng.normal(size=(4, n))
    sc = synth.PlainScene(
        mean=np.stack([(rng.uniform(0, W, n) - W / 2) * z / f, (rng.uniform(0, H, n) - H / 2) * z / f, z]).astype(np.float32),
        scale=np.stack([px[0] * z / f, px[1] * z / f, px[1] * z / f]).astype(np.float32), rot=q.astype(np.float32),
        opacity=rng.uniform(0.05, 0.6, n).astype(np.float32), rgb=rng.uniform(0, 1, (3, n)).astype(np.float32))
    cam = synth.Camera(W, H, f, f, W / 2 - 0.5, H / 2 - 0.5, np.eye(3, 4, dtype=np.float32))
    g = P.gaussians_to_device(sc.arrays())
    rc = P.RenderContext([cam], n, n_feat=0)
    rc.fit(g)
    rc.forward(g)
    torch.cuda.synchronize()
    st, _ = check_binning_self_consistent(rc, "wide rectangles %dx%d n=%d" % (W, H, n))
    assert n < 256 or (st["ntiles"].max() > 64 and ((st["ntiles"] > 0) & (st["ntiles"] <= 16)).any())


@pytest.mark.parametrize("n", [2, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4097])
def test_list_order_at_run_edges(n):
    """One tile's list of n entries, a third of them at equal depths (ordered by
    index): every length at which the sort changes its number of keys per
    thread, its runs or their merging."""
    rng = np.random.default_rng(n)
    z = rng.uniform(2.0, 4.0, n)
    z[rng.permutation(n)[:n // 3]] = 3.0
    q = rng.normal(size=(4, n))
    sc = synth.PlainScene(
        mean=np.stack([rng.uniform(-0.2, 0.2, n), rng.uniform(-0.2, 0.2, n), z]).astype(np.float32),
        scale=rng.uniform(1.5, 4.0, (3, n)).astype(np.float32), rot=q.astype(np.float32),
        opacity=rng.uniform(0.006, 0.02, n).astype(np.float32), rgb=rng.uniform(0, 1, (3, n)).astype(np.float32))
    cam = synth.Camera(16, 16, 20.0, 20.0, 7.5, 7.5, np.eye(3, 4, dtype=np.float32))
    g = P.gaussians_to_device(sc.arrays())
    rc = P.RenderContext([cam], n, n_feat=0)
    rc.fit(g)
    rc.forward(g)
    torch.cuda.synchronize()
    st, _ = check_binning_self_consistent(rc, "one list n=%d" % n)
    assert st["n_isect"] == n


@pytest.mark.parametrize("nf", [0, 16])
@pytest.mark.parametrize("n", [15, 16, 17, 31, 257, 600])
def test_list_parts_of_a_large_view(n, nf):
    """n specks on one tile of a 512x272 view (544 tiles: a round's list in two
    parts, where the one-tile views above take four), some of them opaque
    enough to end pixels inside the second part."""
    rng = np.random.default_rng(100 + n)
    z = rng.uniform(2.0, 4.0, n)
    f = 100.0
    u, v = rng.uniform(242.0, 253.0, n), rng.uniform(130.0, 141.0, n)
    sig = rng.uniform(2.0, 4.0, (3, n))
    o = np.where(rng.uniform(size=n) < 0.1, 0.9, rng.uniform(0.006, 0.03, n))
    q = rng.normal(size=(4, n))
    sc = synth.PlainScene(
        mean=np.stack([(u - 255.5) * z / f, (v - 135.5) * z / f, z]).astype(np.float32),
        scale=(sig * z / f).astype(np.float32), rot=q.astype(np.float32), opacity=o.astype(np.float32),
        rgb=rng.uniform(0, 1, (3, n)).astype(np.float32),
        feat=rng.normal(size=(nf, n)).astype(np.float32) if nf else None)
    cam = synth.Camera(512, 272, f, f, 255.5, 135.5, np.eye(3, 4, dtype=np.float32))
    _check(sc, cam, nf, "large view n=%d nf=%d" % (n, nf), 0.01)


@pytest.mark.parametrize("n", [127, 128, 129, 257, 400])
def test_large_view_among_small_ones(n):
    """A view of 544 tiles renders the same bits alone and between two small
    views (whose workgroups have more waves and longer rounds), and so do
    these."""
    rng = np.random.default_rng(200 + n)
    z = rng.uniform(2.0, 4.0, n)
    f = 100.0
    u, v = rng.uniform(2.0, 13.0, n), rng.uniform(2.0, 13.0, n)
    q = rng.normal(size=(4, n))
    sc = synth.PlainScene(
        mean=np.stack([(u - 7.5) * z / f, (v - 7.5) * z / f, z]).astype(np.float32),
        scale=(rng.uniform(2.0, 4.0, (3, n)) * z / f).astype(np.float32), rot=q.astype(np.float32),
        opacity=np.where(rng.uniform(size=n) < 0.05, 0.9, rng.uniform(0.006, 0.03, n)).astype(np.float32),
        rgb=rng.uniform(0, 1, (3, n)).astype(np.float32))
    pose = np.eye(3, 4, dtype=np.float32)
    cams = [synth.Camera(w, h, f, f, 7.5, 7.5, pose) for w, h in ((16, 16), (512, 272), (40, 24))]
    g = P.gaussians_to_device(sc.arrays())

    def render(cs):
        pix = sum(int(c.width) * int(c.height) for c in cs)
        opts = L.make_opts(0)
        ctx = torch.empty(L.render_ctx_size(cs, n, opts, 64 * n), dtype=torch.uint8, device="cuda")
        out = dict(rgb=torch.zeros(3 * pix, device="cuda"), depth=torch.zeros(pix, device="cuda"),
                   alpha=torch.zeros(pix, device="cuda"))
        L.render_forward(cs, L.make_gaussians(g, n), opts, L.make_images(out), ctx)
        torch.cuda.synchronize()
        return {k: to_np(t) for k, t in out.items()}

    log("case", "large view among small ones n=%d" % n)
    mixed = render(cams)
    at = 0
    for c in cams:
        one, p = render([c]), int(c.width) * int(c.height)
        assert one["alpha"].max() > 0.05
        for k, ch in (("rgb", 3), ("depth", 1), ("alpha", 1)):
            assert np.array_equal(mixed[k][ch * at:ch * (at + p)], one[k]), (c.width, k)
        at += p
