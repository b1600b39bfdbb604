"""Shapes whose records must not end up one after the other on a single
workgroup: the time of the call is held to a few times that of a handful of
short launches, far below that of the serial chain. Results equal the stable
sort."""

import pytest
import torch

from tests.test_gpu_binning_paths import _expected, _records

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qr():
    import paper_2512_20927_amd as qr
    return qr


def _timed(qr, views, tx, ty, capacity):
    """(best time of one call in us, ids, offsets) over a few calls."""
    nv, n = len(views), len(views[0][1])
    rect = torch.cat([v[0] for v in views]).cuda().contiguous()
    depth = torch.cat([v[1] for v in views]).cuda()
    touched = ((rect[:, 2] - rect[:, 0]) * (rect[:, 3] - rect[:, 1])).int().contiguous()
    ws = torch.empty(qr._lib.qr_bin_sort_workspace_size(nv * n, tx, ty * nv, capacity), dtype=torch.uint8, device="cuda")
    gid = torch.empty(capacity, dtype=torch.int32, device="cuda")
    offs = torch.empty(nv * tx * ty + 1, dtype=torch.int32, device="cuda")
    total = torch.empty(1, dtype=torch.int32, device="cuda")
    best = float("inf")
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        qr._lib.qr_bin_sort_views(nv, n, tx, ty, rect, touched, depth, capacity, ws, gid, None, offs, total)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best, gid.cpu().long(), offs.cpu().long()


def _check(views, tx, ty, gid, offs):
    want = [_expected(*v, tx, ty) for v in views]
    base = 0
    for v, (ids, _, o) in enumerate(want):
        assert torch.equal(offs[v * tx * ty:(v + 1) * tx * ty], o[:-1] + base)
        assert torch.equal(gid[base:base + len(ids)], ids)
        base += len(ids)
    assert int(offs[-1]) == base


@pytest.mark.parametrize("nv,n,tx,ty", [(4096, 16, 1, 1), (1024, 16, 2, 2), (64, 64, 4, 4)])
def test_many_small_views_are_taken_side_by_side(qr, nv, n, tx, ty):
    views = [_records(n, tx, ty, 2, v) for v in range(nv)]
    us, gid, offs = _timed(qr, views, tx, ty, 4 * nv * n)
    _check(views, tx, ty, gid, offs)
    assert us <= 300.0, us  # view after view: 2,960 us for 4,096 views, 730 for 1,024


@pytest.mark.parametrize("n,tx,ty,visible,room", [(1_000_000, 81, 61, 1000, 1.0), (1_000_000, 81, 61, 1000, 2.0),
                                                  (200_000, 40, 30, 500, 1.25), (1_000_000, 81, 61, 100_000, 1.25)])
def test_a_small_capacity_leaves_no_long_chunks(qr, n, tx, ty, visible, room):
    """Few visible records of many: the workspace, sized by the pairs, has no
    room for the counts of enough chunks."""
    rect, depth = _records(n, tx, ty, 2, n)
    keep = torch.randperm(n, generator=torch.Generator().manual_seed(visible))[:visible]
    hidden = torch.ones(n, dtype=torch.bool)
    hidden[keep] = False
    rect[hidden] = 0
    pairs = int(((rect[:, 2] - rect[:, 0]) * (rect[:, 3] - rect[:, 1])).sum())
    us, gid, offs = _timed(qr, [(rect, depth)], tx, ty, int(pairs * room))
    _check([(rect, depth)], tx, ty, gid[:pairs], offs)
    assert us <= 150.0, us  # one chunk: 800 us for the first
