"""Lists that the backward walks in segments, at the limits of the rule that
chooses them (64 lists of a view, thresholds of 160 to 1024 entries) and where
a quarter of a tile stops inside a segment, against the FP64 oracle (tolerances
of the render parity tests)."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import log
from tests.test_gpu_blend_edges import _check

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2505_22335_amd as P
    from paper_2505_22335_amd import _lib as L


def _specks(rng, tiles, lens, TX, W, H, nf):
    """lens[i] faint specks inside tile tiles[i] and nowhere else, in depth order at random."""
    tile = np.repeat(tiles, lens)
    n = len(tile)
    f = 100.0
    z = rng.uniform(2.0, 4.0, n)
    u = 16 * (tile % TX) + rng.uniform(5.0, 10.0, n)
    v = 16 * (tile // TX) + rng.uniform(5.0, 10.0, n)
    q = rng.normal(size=(4, n))
    sc = synth.PlainScene(
        mean=np.stack([(u - W / 2 + 0.5) * z / f, (v - H / 2 + 0.5) * z / f, z]).astype(np.float32),
        scale=(rng.uniform(0.8, 1.4, (3, n)) * z / f).astype(np.float32), rot=q.astype(np.float32),
        opacity=rng.uniform(0.006, 0.02, n).astype(np.float32), rgb=rng.uniform(0, 1, (3, n)).astype(np.float32),
        feat=rng.normal(size=(nf, n)).astype(np.float32) if nf else None)
    return sc, synth.Camera(W, H, f, f, W / 2 - 0.5, H / 2 - 0.5, np.eye(3, 4, dtype=np.float32))


@pytest.mark.parametrize("lists,length,nf", [(63, 161, 0), (64, 192, 16), (65, 192, 0), (65, 193, 0), (64, 400, 0),
                                             (65, 1025, 0), (15, 4100, 0), (40, 2100, 0)])
def test_split_slots_used_up(lists, length, nf):
    """Lists of one length in an 80-tile view, the other tiles with 40 entries
    or none: fewer than, as many as and more than the 64 that are split (of 65
    equal ones none is), more than 64 above the last threshold, and long ones
    (most of their entries in the last segment)."""
    rng = np.random.default_rng(lists * 10000 + length)
    TX, TY = 10, 8
    order = rng.permutation(TX * TY)
    lens = np.full(TX * TY, 40 if length < 1000 else 0)
    lens[:lists] = length
    sc, cam = _specks(rng, order, lens, TX, 16 * TX, 16 * TY, nf)
    g = P.gaussians_to_device(sc.arrays())
    rc = P.RenderContext([cam], sc.n, n_feat=nf)
    rc.fit(g)
    rc.forward(g)
    rg = rc.array(L.CTX_TILE_RANGE, torch.int32, width=2).cpu().numpy()
    got = np.sort(rg[:, 1] - rg[:, 0])
    log("case split slots", lists, length, nf, "lists", got[-lists], "to", got[-1])
    assert np.array_equal(got, np.sort(lens))
    _check(sc, cam, nf, "split slots %d of %d" % (lists, length), 0.15)


@pytest.mark.parametrize("W,H,tx,ty", [(16, 16, 0, 0), (512, 272, 15, 8)])
@pytest.mark.parametrize("nf", [0, 16])
@pytest.mark.parametrize("at", [5, 100, 140, 230, 270, 390])
def test_quarter_stops_in_a_segment(at, nf, W, H, tx, ty):
    """A list of 900 entries (segments of 128, the last of 516) over one tile of
    a small and of a large view; its upper left quarter is closed by opaque
    entries from position at on: inside the first, second, third and last
    segment, and across their ends. The quarter records no state at later
    boundaries, and the other quarters go on past them."""
    n = 900
    rng = np.random.default_rng(at + nf)
    z = np.linspace(2.0, 4.0, n)
    u, v = rng.uniform(-0.5, 15.5, n), rng.uniform(-0.5, 15.5, n)
    sig, o = rng.uniform(1.0, 2.0, n), rng.uniform(0.006, 0.03, n)
    k = np.arange(60)
    u[at:at + 60], v[at:at + 60] = 2.0 + 3.0 * (k & 1), 2.0 + 3.0 * ((k >> 1) & 1)
    sig[at:at + 60], o[at:at + 60] = 2.0, 0.9
    f, cx, cy = 20.0, 7.5 + 16 * tx, 7.5 + 16 * ty
    sc = synth.PlainScene(
        mean=np.stack([(u - 7.5) * z / f, (v - 7.5) * z / f, z]).astype(np.float32),
        scale=np.broadcast_to(sig * z / f, (3, n)).astype(np.float32),
        rot=np.broadcast_to(np.array([1.0, 0.0, 0.0, 0.0])[:, None], (4, n)).astype(np.float32),
        opacity=o.astype(np.float32), rgb=rng.uniform(0, 1, (3, n)).astype(np.float32),
        feat=rng.normal(size=(nf, n)).astype(np.float32) if nf else None)
    cam = synth.Camera(W, H, f, f, cx, cy, np.eye(3, 4, dtype=np.float32))
    # the specks are round: no gradient reaches their rotation
    _check(sc, cam, nf, "quarter stops at %d nf=%d %dx%d" % (at, nf, W, H), 0.15, ("mean", "scale", "opacity", "rgb"))


@pytest.mark.parametrize("lists", [64, 65])
def test_splits_are_the_views_own(lists):
    """A view with 64 or 65 long lists gives the same bits alone and beside a
    view with others, images and gradients."""
    rng = np.random.default_rng(lists)
    TX, TY = 10, 8
    lens = np.full(TX * TY, 30)
    lens[:lists] = 300
    sc, cam = _specks(rng, rng.permutation(TX * TY), lens, TX, 16 * TX, 16 * TY, 0)
    other = synth.Camera(160, 128, 60.0, 60.0, 79.5, 63.5, np.eye(3, 4, dtype=np.float32))
    g = P.gaussians_to_device(sc.arrays())
    d = {f: torch.as_tensor(rng.normal(size=(1, 3, 128, 160) if f == "rgb" else (1, 128, 160)).astype(np.float32)).cuda()
         for f in ("rgb", "depth", "alpha")}

    def both(cams, up):
        rc = P.RenderContext(cams, sc.n, n_feat=0)
        rc.fit(g)
        img = rc.forward(g)
        dg, _ = rc.backward(g, up)
        torch.cuda.synchronize()
        return img, dg

    log("case splits alone and in a batch", lists)
    i1, g1 = both([cam], d)
    i2, g2 = both([other, cam], {k: torch.cat([v, v]) for k, v in d.items()})
    assert all(torch.equal(i1[k][0], i2[k][1]) for k in i1)
    assert all(torch.equal(g1[k][0], g2[k][1]) for k in g1), [k for k in g1 if not torch.equal(g1[k][0], g2[k][1])]
