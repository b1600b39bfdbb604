"""Groups of four pixels with more distinct selections than the renderer keeps
in one walk (32): they are collected in further walks, two groups of a wave at
a time. Maps, T^Q and selections against the FP64 oracle, batched bit-identical
to single-view, at the widths with their own gather and for both rules that
collect groups; the same at K where no group can exceed the capacity."""

import numpy as np
import pytest
import torch

import oracle
from tests.parity_util import DECISION_WINDOW, FP32_TOL, proj_for_oracle
from tests.test_gpu_backward import _setup
from tests.test_gpu_backward_slots import _scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20927_amd as qr
    return qr


@pytest.mark.parametrize("rule,K,dim,storage,bf16_out", [
    ("quantile", 8, 48, "f32", False), ("quantile", 9, 16, "f32", False), ("quantile", 64, 16, "bf16", False),
    ("quantile", 64, 144, "f32", False), ("quantile", 40, 528, "fp8", False), ("quantile", 64, 144, "f32", True),
    ("stratified", 64, 48, "f32", False), ("stratified", 64, 512, "bf16", False)])
def test_group_capacity(qr, rule, K, dim, storage, bf16_out):
    L = qr._lib
    sc, cam = _scene(9000, 40, dim, False)
    sc.opacity[:9000] *= 0.4  # many selections before a ray saturates
    W, H = cam.width, cam.height
    pr, bins, feats, scale, host, dec = _setup(qr, sc, cam, storage)
    prm = qr.RenderParams(selection=L.QR_SELECT_STRATIFIED if rule == "stratified" else L.QR_SELECT_QUANTILE,
                          out_dtype=L.QR_BF16 if bf16_out else L.QR_F32)
    r = qr.render_quantile(pr, bins, feats, W, H, K, prm, scale, debug=True)
    torch.cuda.synchronize()
    sel = r["sel_gid"].cpu().numpy()
    over = [len(set(sel[y, x:x + 4].ravel()) - {-1}) > 32 for y in range(H) for x in range(0, W, 4)]
    if K >= 40:
        assert sum(over) > 8  # several groups of one wave among them
    proj = proj_for_oracle(host["pr"])
    render = oracle.render_stratified if rule == "stratified" else oracle.render_quantile
    o = render(proj, host["gids"], host["offs"], dec, W, H, K)
    clean = o["margin"] > DECISION_WINDOW
    assert clean.mean() > 0.5
    got = r["out"].float().cpu().numpy().astype(np.float64)
    err = np.linalg.norm(got - o["out"], axis=-1) / np.maximum(np.linalg.norm(o["out"], axis=-1), 1e-6)
    # float32 maps: the parity tolerance; bfloat16 maps: half an ulp of 8 bits besides
    assert err[clean].max() <= FP32_TOL + (2.0 ** -8 if bf16_out else 0.0)
    n = r["n_sel"].cpu().numpy()
    assert np.array_equal(n[clean], np.asarray(o["n_sel"])[clean])
    assert np.array_equal((sel >= 0).sum(-1), n)
    np.testing.assert_allclose(r["T_q"].cpu().numpy()[clean], np.asarray(o["T_q"])[clean], rtol=1e-4, atol=1e-6)
    # the batched launches render the same bits
    from paper_2512_20927_amd.batched import BatchedQuantile
    out = torch.empty_like(r["out"])
    bq = BatchedQuantile([dict(tile_offsets=bins.tile_offsets, sorted_gid=bins.sorted_gid, means2d=pr.means2d,
                               conic_opacity=pr.conic_opacity, features=feats, feature_scale=scale, out=out,
                               width=W, height=H)], K, dim, L.DTYPE_CODE[feats.dtype], prm.c())
    for per_cu in (0, 2):
        out.zero_()
        bq.render("natural", per_cu)
        assert torch.equal(out, r["out"])
