"""The Q-Render backward where a tile's distinct selections take several passes
of 32 slots, run out of slots (256) or lie past the slot bitmap (list position
8,192), at the widths where the waves share columns differently and at the K
where the workgroup's shape changes (20, 48). Compared with the FP64 oracle
under test_gpu_backward's element-wise bound."""

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity_util import DECISION_WINDOW, proj_for_oracle
from tests.test_gpu_backward import _compare, _setup, _t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20927_amd as qr
    return qr


def _scene(n_small, n_big, dim, corner):
    """Gaussians of about a pixel, over the whole 30 x 26 picture or (corner)
    on a few of its pixels, in front of large ones."""
    rng = np.random.default_rng(n_small + dim)
    n = n_small + n_big
    means = np.zeros((n, 3), np.float32)
    lo, hi = (-0.97, -0.90) if corner else (-1.2, 1.2)
    means[:n_small, :2] = rng.uniform(lo, hi, (n_small, 2))
    means[:n_small, 2] = -1.0 + rng.uniform(0.0, 0.01, n_small)
    means[n_small:, :2] = rng.uniform(-2.0, 2.0, (n_big, 2))
    means[n_small:, 2] = 1.0 + rng.uniform(0.0, 0.5, n_big)
    scales = np.concatenate([np.full((n_small, 3), 0.004, np.float32),
                             rng.uniform(0.15, 0.4, (n_big, 3)).astype(np.float32)])
    quats = rng.standard_normal((n, 4)).astype(np.float32)
    opacity = np.concatenate([rng.uniform(0.3, 0.9, n_small), rng.uniform(0.3, 0.7, n_big)]).astype(np.float32)
    cam = synth.tiny_camera(30)
    cam.height, cam.cy = 26, 13.0
    return synth.Scene(means, scales, quats, opacity, rng.standard_normal((n, dim)).astype(np.float32)), cam


@pytest.mark.parametrize("K,dim,storage,n_small,corner", [
    (1, 16, "f32", 300, False), (8, 32, "f32", 300, False), (20, 48, "bf16", 900, False),
    (21, 144, "fp8", 900, False), (48, 272, "f32", 2400, False), (49, 512, "f32", 2400, False),
    (8, 528, "bf16", 2400, False), (64, 1040, "fp8", 300, False), (8, 16, "f32", 8300, True)])
def test_slots(qr, K, dim, storage, n_small, corner):
    sc, cam = _scene(n_small, 40, dim, corner)
    W, H = cam.width, cam.height
    pr, bins, feats, scale, host, dec = _setup(qr, sc, cam, storage)
    proj = proj_for_oracle(host["pr"])
    fw = oracle.render_quantile(proj, host["gids"], host["offs"], dec, W, H, K)
    g = np.random.default_rng(K).standard_normal((H, W, dim)) * (fw["margin"] > DECISION_WINDOW)[..., None]
    gf, gm, gc = (torch.zeros(sc.n, k, device="cuda") for k in (dim, 2, 4))
    qr._lib.qr_render_quantile_backward(W, H, qr.RenderParams().c(), K, bins.tile_offsets, bins.sorted_gid,
                                        pr.means2d, pr.conic_opacity, feats, scale,
                                        _t(g.astype(np.float32)), gf, gm, gc)
    # the oracle differentiates what the kernel was given: the float32 gradient
    orc = oracle.quantile_backward(proj, host["gids"], host["offs"], dec, W, H, K,
                                   g.astype(np.float32).astype(np.float64), magnitude=True)
    _compare(dict(gf=gf.cpu().numpy(), gm=gm.cpu().numpy(), gc=gc.cpu().numpy()), orc)
