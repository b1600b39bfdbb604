"""dL/d(out) that is not finite at a few values, in tiles with more distinct
selections than the first 32 slots: the later ones take it from their own
pixels only, and other columns than the values' take nothing of it.

Compared with the same call on zeros at those values. The two differ by the
order of at most 16 float atomics of an entry (tiles and column shares), so by
2^-20 of the magnitude of its terms, which is the call on |dL/d(out)| for the
feature gradients (their weights are not negative); the bound is twice that."""

import numpy as np
import pytest
import torch

from tests.test_gpu_backward import _setup, _t
from tests.test_gpu_backward_slots import _scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20927_amd as qr
    return qr


@pytest.mark.parametrize("K,dim,storage", [(20, 48, "f32"), (8, 144, "fp8"), (48, 80, "f32"), (48, 272, "bf16"),
                                           (49, 512, "f32"), (8, 528, "f32"), (64, 16, "bf16")])
def test_later_slots_take_their_own_pixels_only(qr, K, dim, storage):
    sc, cam = _scene(900, 40, dim, False)
    W, H = cam.width, cam.height
    pr, bins, feats, scale, host, _ = _setup(qr, sc, cam, storage)
    sel = qr.render_quantile(pr, bins, feats, W, H, K, feature_scale=scale, debug=True)["sel_gid"]
    sel = sel.cpu().numpy().reshape(H, W, K)
    offs, gids = host["offs"].ravel(), host["gids"].ravel()
    g0 = np.random.default_rng(K).standard_normal((H, W, dim)).astype(np.float32)
    cols = np.arange(1, dim, 7)
    bad = np.zeros((H, W), bool)
    first = np.zeros(sc.n, bool)  # among the first 32 slots of a tile
    tx = (W + 15) // 16
    for t in range(tx * ((H + 15) // 16)):
        y, x = t // tx * 16, t % tx * 16
        ids = np.unique(sel[y:y + 16, x:x + 16])
        ids = ids[ids >= 0]
        assert ids.size > 64
        lst = gids[offs[t]:offs[t + 1]]
        first[lst[np.isin(lst, ids)][:32]] = True
        bad[y + 3, x + 5] = bad[min(y + 9, H - 1), min(x + 15, W - 1)] = True
    g0[bad] = 0.0
    g = g0.copy()
    ys, xs = np.nonzero(bad)
    for k, (y, x) in enumerate(zip(ys, xs)):
        g[y, x, cols] = (np.inf, -np.inf, np.nan)[k % 3]

    def run(grad):
        gf, gm, gc = (torch.zeros(sc.n, k, device="cuda") for k in (dim, 2, 4))
        qr._lib.qr_render_quantile_backward(W, H, qr.RenderParams().c(), K, bins.tile_offsets, bins.sorted_gid,
                                            pr.means2d, pr.conic_opacity, feats, scale, _t(grad), gf, gm, gc)
        return gf.cpu().numpy(), gm.cpu().numpy(), gc.cpu().numpy()

    gf, gm, gc = run(g)
    wf, wm, wc = run(g0)
    mag = run(np.abs(g0))[0]
    hit = np.zeros(sc.n, bool)  # selected where the gradient is not finite
    hit[np.unique(sel[bad][sel[bad] >= 0])] = True
    close = np.abs(gf - wf) <= 2.0 ** -19 * mag + 1e-30
    other = np.setdiff1d(np.arange(dim), cols)
    assert close[:, other].all()
    assert (~hit & ~first).sum() > 64 and close[~hit & ~first].all()
    assert not np.isfinite(gf[hit][:, cols]).any()
    assert np.isfinite(gm[~hit]).all() and np.isfinite(gc[~hit]).all()
    assert not np.isfinite(gc[hit]).all()
