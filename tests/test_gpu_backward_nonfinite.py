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


@pytest.mark.parametrize("near", [0, 6])
@pytest.mark.parametrize("K,dim", [(3, 64), (24, 144), (4, 512), (50, 528)])
def test_selections_far_down_the_list_take_their_own_pixels_only(qr, K, dim, near):
    """The same past list position 2,048, with and without selections before it."""
    rng = np.random.default_rng(dim + K)
    n, fill = 25, 2048  # Gaussian 0 fills the list; pairs of small ones lie over the tile
    spots = np.stack(np.meshgrid([2.5, 6.5, 10.5, 14.5], [3.0, 8.0, 13.0]), -1).reshape(-1, 2)
    means = np.concatenate([[[8.0, 8.0]], np.repeat(spots, 2, 0) + rng.uniform(-0.6, 0.6, (24, 2))]).astype(np.float32)
    co = np.tile(np.float32([0.8, 0.1, 0.9, 0.0]), (n, 1))
    co[1:, 3] = rng.uniform(0.5, 0.9, n - 1)
    ids = np.concatenate([1 + np.arange(near), np.zeros(fill - near, int), 1 + near + np.arange(n - 1 - near)])
    offs, gid = _t(np.int32([0, len(ids)])), _t(ids.astype(np.int32))
    m, c, feats = _t(means), _t(co), _t(rng.standard_normal((n, dim)).astype(np.float32))
    prm = qr.RenderParams()
    r = qr.render_quantile(qr.Projected(m, c, None, None, None), qr.Bins(offs, gid, None, len(ids)), feats, 16, 16, K,
                           prm, debug=True)
    sel = r["sel_gid"].view(256, K).cpu().numpy()
    cols = np.arange(1, dim, 7)
    bad = [16 * 13 + 14, 16 * 12 + 14]  # two pixels near the last spot
    g0 = rng.standard_normal((256, dim)).astype(np.float32)
    g0[bad] = 0.0
    g = g0.copy()
    g[bad[0], cols], g[bad[1], cols] = np.inf, np.nan

    def run(grad):
        gf, gm, gc = (torch.zeros(n, k, device="cuda") for k in (dim, 2, 4))
        qr._lib.qr_render_quantile_backward(16, 16, prm.c(), K, offs, gid, m, c, feats, None,
                                            _t(grad.reshape(16, 16, dim)), gf, gm, gc)
        return gf.cpu().numpy()

    gf, want, mag = run(g), run(g0), run(np.abs(g0))
    hit = np.isin(np.arange(n), sel[bad][sel[bad] >= 0])
    far = np.arange(n) > near
    assert (far & hit).any() and (far & ~hit).sum() > 8
    close = np.abs(gf - want) <= 2.0 ** -19 * mag + 1e-30
    assert close[:, np.setdiff1d(np.arange(dim), cols)].all() and close[far & ~hit].all()
    assert not np.isfinite(gf[far & hit][:, cols]).any()
