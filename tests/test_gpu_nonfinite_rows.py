"""A feature row that is not finite reaches the pixels that selected it and no
other: four neighbouring pixels share the rows that any of them selected, with
weight 0 where a pixel did not. Narrow and wide maps, every stored type of
float; compared bit for bit with the same table whose bad rows are zero."""

import pytest
import torch

from tests.test_gpu_backward import _setup
from tests.test_gpu_backward_slots import _scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20927_amd as qr
    return qr


@pytest.mark.parametrize("rule,K", [("quantile", 5), ("quantile", 16), ("quantile", 64), ("stratified", 24),
                                    ("topk", 4)])
@pytest.mark.parametrize("dim,storage", [(16, "f32"), (48, "bf16"), (128, "f32"), (144, "f32")])
def test_other_pixels_stay_as_they_are(qr, rule, K, dim, storage):
    L = qr._lib
    sc, cam = _scene(9000, 40, dim, False)
    sc.opacity[:9000] *= 0.4  # many selections before a ray saturates
    W, H = cam.width, cam.height
    pr, bins, feats, _, _, _ = _setup(qr, sc, cam, storage)
    prm = qr.RenderParams(selection=dict(quantile=L.QR_SELECT_QUANTILE, stratified=L.QR_SELECT_STRATIFIED,
                                         topk=L.QR_SELECT_TOPK)[rule])
    bad = torch.arange(0, sc.n, 23, device="cuda")
    zero = feats.clone()
    zero[bad] = 0
    feats[bad] = float("inf")
    feats[bad[::2], ::3] = float("nan")
    r = qr.render_quantile(pr, bins, feats, W, H, K, prm, debug=True)
    want = qr.render_quantile(pr, bins, zero, W, H, K, prm)["out"]
    hit = (torch.isin(r["sel_gid"], bad.int()) & (r["sel_gid"] >= 0)).any(-1)
    assert 20 < int(hit.sum()) < W * H - 20
    assert torch.equal(r["out"][~hit], want[~hit])
    assert not bool(torch.isfinite(r["out"][hit]).all(-1).any())
