"""Plain renders and their gradients against recorded values.

The gradients of scale and rotation come from second moments that are FP32
sums of terms far larger than their result: a change of the last bits of the
transmittance, of the order of a sum or of where a list is cut moves single
elements by up to 1e-3 of the gradient's rms, which no comparison within the
oracle's tolerances shows. The recorded values are those of the kernels that
walked a list in rounds of 256 entries (128 where it is split) and two halves.
Bound per element: 2^-20 of max(rms, |value|), sixteen roundings of the
result, none of the terms; the forward's state is the same to the bit."""
import os

import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import log, to_np, upstream

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2505_22335_amd as P
    from paper_2505_22335_amd import _lib as L

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "render_recorded.npz")
FIELDS = ("mean", "scale", "rot", "opacity", "rgb")


def scene(W, H):
    """1200 Gaussians over a 64x48 patch of a W x H view, two thirds of them in a
    corner of it, specks and blobs, faint and opaque: lists from a hundred entries
    to several hundred, many pixels stopped."""
    n = 1200
    rng = np.random.default_rng(77)
    z = rng.uniform(1.0, 4.0, n)
    f = 200.0
    u, v = rng.uniform(-4.0, 68.0, n), rng.uniform(-4.0, 52.0, n)
    u[::3], v[::3] = rng.uniform(0.0, 28.0, n // 3), rng.uniform(0.0, 28.0, n // 3)
    u[1::3], v[1::3] = rng.uniform(0.0, 28.0, n // 3), rng.uniform(0.0, 28.0, n // 3)
    sig = np.exp(rng.uniform(np.log(1.0), np.log(4.0), (3, n)))
    sig[:, :60] *= 4.0
    q = rng.normal(size=(4, n))
    sc = synth.PlainScene(
        mean=np.stack([(u - 31.5) * z / f, (v - 23.5) * z / f, z]).astype(np.float32),
        scale=(sig * z / f).astype(np.float32), rot=(q / np.linalg.norm(q, axis=0)).astype(np.float32),
        opacity=np.where(np.arange(n) % 4 == 0, rng.uniform(0.3, 0.95, n), rng.uniform(0.006, 0.1, n)).astype(np.float32),
        rgb=rng.uniform(0, 1, (3, n)).astype(np.float32))
    return sc, synth.Camera(W, H, f, f, 31.5, 23.5, np.eye(3, 4, dtype=np.float32))


def render(W, H):
    sc, cam = scene(W, H)
    g = P.gaussians_to_device(sc.arrays())
    rc = P.RenderContext([cam], sc.n, n_feat=0)
    rc.fit(g)
    rc.forward(g)
    G = upstream(5, H, W, 0)
    dg, _ = rc.backward(g, {k: torch.as_tensor(v[None].astype(np.float32)).cuda() for k, v in G.items()})
    torch.cuda.synchronize()
    out = {k: to_np(dg[k][0]) for k in FIELDS}
    out["tfinal"] = rc.array(L.CTX_TFINAL, torch.float32).cpu().numpy().reshape(H, W)[:48, :64]
    out["ncontrib"] = rc.array(L.CTX_NCONTRIB, torch.int32).cpu().numpy().reshape(H, W)[:48, :64]
    rg = rc.array(L.CTX_TILE_RANGE, torch.int32, width=2).cpu().numpy()
    return out, rg[:, 1] - rg[:, 0]


@pytest.mark.parametrize("W,H", [(64, 48), (528, 272)])
def test_render_equals_recorded(W, H):
    """A small view and one of more than 512 tiles: T and the last
    contributors as recorded, every gradient within 2^-20."""
    rec = np.load(GOLDEN)
    out, lens = render(W, H)
    log("case recorded %dx%d" % (W, H), "lists of", int(lens.min()), "to", int(lens.max()), "split", int((lens > 160).sum()))
    assert (lens > 256).any() and ((lens > 0) & (lens <= 160)).any()
    for k in ("tfinal", "ncontrib"):
        assert np.array_equal(out[k], rec["%dx%d_%s" % (W, H, k)]), k
    for k in FIELDS:
        x, y = out[k].astype(np.float64), rec["%dx%d_%s" % (W, H, k)].astype(np.float64)
        d = np.abs(x - y) / np.maximum(np.sqrt((y ** 2).mean()), np.abs(y))
        log("   %s largest move %.2e" % (k, d.max()))
        assert d.max() <= 2.0 ** -20, (k, d.max())
