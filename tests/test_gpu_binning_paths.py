"""Binning by counters in LDS (one workgroup for small scenes, chunks of
records for larger ones), by counters in global memory, and the register sort:
offsets, ids and keys equal the stable sort by (tile, depth, id) of the same
records, at the sizes where one gives way to the next."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qr():
    import paper_2512_20927_amd as qr
    return qr


def _records(n, tx, ty, span, seed):
    """n records of one view: rectangles of up to `span` tiles a side (some
    empty), depths with ties (ties are ordered by id)."""
    g = torch.Generator().manual_seed(seed)
    x0 = torch.randint(0, tx, (n,), generator=g)
    y0 = torch.randint(0, ty, (n,), generator=g)
    x1 = (x0 + torch.randint(0, span + 1, (n,), generator=g)).clamp(max=tx)
    y1 = (y0 + torch.randint(1, span + 1, (n,), generator=g)).clamp(max=ty)
    depth = torch.randint(1, max(n // 2, 2), (n,), generator=g).float() / 7
    return torch.stack([x0, y0, x1, y1], 1).int(), depth


def _expected(rect, depth, tx, ty):
    r = rect.long()
    w, h = r[:, 2] - r[:, 0], r[:, 3] - r[:, 1]
    count = w * h
    gid = torch.repeat_interleave(torch.arange(len(r)), count)
    k = torch.arange(int(count.sum())) - torch.repeat_interleave(count.cumsum(0) - count, count)
    tile = (r[gid, 1] + k // w[gid]) * tx + r[gid, 0] + k % w[gid]
    bits = depth.view(torch.int32).long()[gid]
    order = torch.argsort(bits, stable=True)
    order = order[torch.argsort(tile[order], stable=True)]
    offs = torch.zeros(tx * ty + 1, dtype=torch.long)
    offs[1:] = torch.bincount(tile, minlength=tx * ty).cumsum(0)
    return gid[order], (tile[order] << 32) | bits[order], offs


def _run(qr, views, tx, ty, capacity):
    import ctypes
    from paper_2512_20927_amd import _lib
    lib = _lib.lib()
    rect = torch.cat([v[0] for v in views]).cuda().contiguous()
    depth = torch.cat([v[1] for v in views]).cuda()
    touched = ((rect[:, 2] - rect[:, 0]) * (rect[:, 3] - rect[:, 1])).int().contiguous()
    nv, n = len(views), len(views[0][1])
    size = ctypes.c_size_t()
    assert lib.qr_bin_sort_workspace_size(nv * n, tx, ty * nv, capacity, ctypes.byref(size)) == 0
    ws = torch.empty(size.value, dtype=torch.uint8, device="cuda")
    gids = torch.full((max(capacity, 1),), -1, dtype=torch.int32, device="cuda")
    keys = torch.zeros(max(capacity, 1), dtype=torch.int64, device="cuda")
    offs = torch.empty(nv * tx * ty + 1, dtype=torch.int32, device="cuda")
    total = torch.empty(1, dtype=torch.int32, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = lib.qr_bin_sort_views(ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), nv, n, tx, ty, p(rect),
                               p(touched), p(depth), capacity, p(ws), size, p(gids), p(keys), p(offs), p(total))
    assert rc == 0
    torch.cuda.synchronize()
    return gids.cpu().long(), keys.cpu(), offs.cpu().long(), int(total)


SHAPES = [  # n_views, n, tiles_x, tiles_y, span
    (1, 1, 1, 1, 1), (1, 64, 1, 1, 1), (1, 65, 1, 1, 1), (1, 257, 1, 1, 1), (1, 513, 1, 1, 1),
    (1, 1025, 1, 1, 1), (1, 2048, 1, 1, 1), (1, 2049, 1, 1, 1),
    (1, 1000, 4, 4, 3), (3, 700, 9, 7, 4),      # one workgroup
    (1, 16, 64, 64, 30), (1, 17, 64, 64, 30),   # its limit: 2^16 records times tiles, 4096 tiles
    (2, 50, 64, 33, 20),
    (1, 5000, 21, 16, 3), (3, 2500, 13, 11, 5), (1, 300_000, 30, 20, 1), (200, 90, 50, 10, 6),  # chunks
    (1, 400, 128, 128, 40), (1, 400, 129, 128, 40),  # 16384 tiles in LDS and one more row
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_offsets_ids_and_keys_equal_the_stable_sort(qr, shape):
    nv, n, tx, ty, span = shape
    views = [_records(n, tx, ty, span, 31 * n + v) for v in range(nv)]
    want = [_expected(*v, tx, ty) for v in views]
    total = sum(len(w[0]) for w in want)
    base, offs_w = 0, []
    for v, w in enumerate(want):
        offs_w.append(w[2][:-1] + base)
        base += len(w[0])
    offs_w = torch.cat(offs_w + [torch.tensor([base])])
    gid_w = torch.cat([w[0] for w in want])
    key_w = torch.cat([w[1] + (v * tx * ty << 32) for v, w in enumerate(want)])
    # room for the chunks' counts (8 bytes a pair hold two) or not: both orders
    # of the buckets end in the same sort
    for capacity in {total, max(total, nv * tx * ty * 200 // 2)}:
        gids, keys, offs, got = _run(qr, views, tx, ty, capacity)
        assert got == total
        assert torch.equal(offs, offs_w)
        assert torch.equal(gids[:total], gid_w)
        assert torch.equal(keys[:total], key_w)


@pytest.mark.parametrize("shape", [(1, 1000, 4, 4, 3), (2, 3000, 40, 30, 4)], ids=["one", "chunks"])
@pytest.mark.parametrize("part", [0, 1, 2], ids=["none", "half", "less_one"])
def test_a_capacity_that_is_too_small_is_reported(qr, shape, part):
    nv, n, tx, ty, span = shape
    views = [_records(n, tx, ty, span, 7 + v) for v in range(nv)]
    want = [_expected(*v, tx, ty) for v in views]
    total = sum(len(w[0]) for w in want)
    _, _, offs, got = _run(qr, views, tx, ty, [0, total // 2, total - 1][part])
    assert got == total and int(offs[-1]) == total
