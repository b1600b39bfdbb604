"""Scenes of pixel-sized, faint Gaussians, where most groups of four pixels select
more distinct Gaussians than the renderer keeps in one walk: float32 maps take
them in parts, bfloat16 maps in further walks. The two agree, and the parts do
not cost a walk of the whole list each."""

import pytest
import torch

pytestmark = pytest.mark.gpu
W, H = 320, 240


@pytest.fixture(scope="module")
def qr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20927_amd as qr
    return qr


@pytest.fixture(scope="module")
def scene(qr):
    n = 750_000
    g = torch.Generator("cuda").manual_seed(3)
    r = lambda *s: torch.rand(*s, generator=g, device="cuda")  # noqa: E731
    mean = r(n, 2) * torch.tensor([W, H], device="cuda")
    var = 0.3 + (r(n) * 0.35) ** 2
    o = 0.02 + 0.08 * r(n)
    rad = torch.sqrt(2 * torch.log(o * 255).clamp(min=0) * var)
    t = torch.tensor([W - 1, H - 1], device="cuda")
    lo = (mean - rad[:, None] - .5).ceil().clamp(min=0).minimum(t) // 16
    hi = (mean + rad[:, None] - .5).floor().clamp(min=0).minimum(t) // 16 + 1
    rect = torch.cat([lo, hi], 1).int().contiguous()
    pr = qr.Projected(mean.contiguous(), torch.stack([1 / var, 0 * var, 1 / var, o], 1).contiguous(), r(n) * 3 + 1, rect,
                      ((rect[:, 2] - rect[:, 0]) * (rect[:, 3] - rect[:, 1])).int().contiguous())
    return pr, qr.bin_sort(pr, W, H)


@pytest.mark.parametrize("rule", ["QR_SELECT_QUANTILE", "QR_SELECT_STRATIFIED"])
@pytest.mark.parametrize("K,dim,storage", [(9, 16, torch.float32), (16, 48, torch.bfloat16), (40, 128, torch.float32),
                                           (64, 528, torch.bfloat16)])
def test_parts_and_further_walks_agree(qr, scene, rule, K, dim, storage):
    L = qr._lib
    pr, bins = scene
    f = torch.randn(pr.depth.numel(), dim, device="cuda", generator=torch.Generator("cuda").manual_seed(K)).to(storage)
    rule = getattr(L, rule)
    a = qr.render_quantile(pr, bins, f, W, H, K, qr.RenderParams(selection=rule), debug=True)
    b = qr.render_quantile(pr, bins, f, W, H, K, qr.RenderParams(selection=rule, out_dtype=L.QR_BF16), debug=True)
    for k in ("T_q", "n_sel", "sel_gid", "sel_w"):
        assert torch.equal(a[k], b[k])
    g = a["sel_gid"].view(H, W // 4, 4 * K).sort(-1).values
    distinct = ((g[..., 1:] != g[..., :-1]) & (g[..., 1:] >= 0)).sum(-1) + (g[..., 0] >= 0)
    if K > 9:  # (K = 9: the first K whose groups could)
        assert (distinct > 32).float().mean() > 0.3
    # half an ulp of bfloat16's eight bits, and the two orders of float32 sums of n terms: the row of largest magnitude
    # among the selected bounds them
    x, y = a["out"].double(), b["out"].double()
    big = f.abs().amax().double() * K * 2.0 ** -22
    assert bool(((x - y).abs() <= x.abs() * 2.0 ** -8 + big).all())


def test_parts_cost_less_than_walks(qr, scene):
    pr, bins = scene
    f = torch.randn(pr.depth.numel(), 16, device="cuda")
    out = torch.empty(H, W, 16, device="cuda")

    def best(K):
        us = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            qr.render_quantile(pr, bins, f, W, H, K, out=out)
            b.record()
            b.synchronize()
            us.append(a.elapsed_time(b))
        return min(us)
    # K = 8 takes one walk; further walks of the whole list for two groups of a wave at a time took six times as long
    assert best(16) <= 3.0 * best(8)
