"""The FP32 sums of the decoder backward over the views of a call: their
rounding stays that of a few views, however many a call has."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import log
from tests.test_gpu_decode import _cams_tiny, _oracle_decode

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2505_22335_amd as P
    from paper_2505_22335_amd.pipeline import anchors_to_device


def _error(sc, cams, grads, in_dim):
    """Norm of the error of d_params against the FP64 oracle over the oracle's norm."""
    a = anchors_to_device(sc)
    dec = P.Decoder(a.A, sc.k, 16, 0, a.l_o, a.l_s, in_dim=in_dim)
    dg = {f: torch.as_tensor(np.stack([g[f] for g in grads]).astype(np.float32)).cuda() for f in grads[0]}
    _, _, _, d_params = dec.backward(a.xyz, a.feat, a.off, a.params, cams, dg)
    torch.cuda.synchronize()
    _, ref = _oracle_decode(sc, cams, grads)
    parts = []
    for name in ("opacity", "rgb", "scale", "rot", "feat"):
        w = ref["weights"][name]
        parts += [w["W1"][:, :35].ravel(), w["b1"].ravel(), w["W2"].ravel(), w["b2"].ravel(), w["W1"][:, 35:].ravel()]
    r = np.concatenate(parts)
    return float(np.linalg.norm(d_params.double().cpu().numpy() - r) / np.linalg.norm(r))


@pytest.mark.parametrize("A,nv,k,in_dim", [(300, 16, 10, 38), (300, 64, 5, 35), (4500, 6, 10, 36), (300, 16, 16, 36)])
def test_error_does_not_grow_with_the_views(A, nv, k, in_dim):
    """Against FP64, at most 1.5 times the error of one view's gradients. A
    chain of m FP32 sums of terms of random sign is 2^-24 sqrt(m / 6) of its
    norm away: 7e-8 for four items and the four to sixteen sums of such
    chunks, beside the 1.1e-7 of the items themselves (1.2 times); over sixteen
    views of four sums an item it would be 2e-7 (twice)."""
    sc = synth.tiny_anchor_scene(9, A, k=k, n_feat=16, in_dim=in_dim)
    cams = _cams_tiny(nv)
    rng = np.random.default_rng(A + nv)
    n = A * k
    grads = [{f: rng.normal(size=(m, n) if m > 1 else n).astype(np.float32)
              for f, m in (("mean", 3), ("scale", 3), ("rot", 4), ("opacity", 1), ("rgb", 3), ("feat", 16))}
             for _ in range(nv)]
    one = np.mean([_error(sc, [cams[v]], [grads[v]], in_dim) for v in range(3)])
    all_ = _error(sc, cams, grads, in_dim)
    log("case view sums A=%d views=%d k=%d in_dim=%d: one view %.2e all %.2e" % (A, nv, k, in_dim, one, all_))
    assert all_ <= 1.5 * one
