"""The scenes of test_gpu_backward_slots reach what they are there for: tiles
with more distinct selections than a pass has slots (32), than a tile has (256),
and selections past the slot bitmap (list position 8,192)."""

import numpy as np
import pytest
import torch

from tests import test_gpu_backward_slots as slots
from tests.test_gpu_backward import _setup

pytestmark = pytest.mark.gpu

CASES = next(m for m in slots.test_slots.pytestmark if m.name == "parametrize").args[1]


def _tiles(case):
    """(distinct selections, largest selected list position) of every tile."""
    import paper_2512_20927_amd as qr
    K, dim, storage, n_small, corner = case
    sc, cam = slots._scene(n_small, 40, dim, corner)
    pr, bins, feats, _, host, _ = _setup(qr, sc, cam, "f32")
    out = qr.render_quantile(pr, bins, feats, cam.width, cam.height, K, debug=True)
    sel = out["sel_gid"].cpu().numpy().reshape(cam.height, cam.width, K)
    offs, gids = np.asarray(host["offs"]).ravel(), np.asarray(host["gids"]).ravel()
    tx = (cam.width + 15) // 16
    res = []
    for t in range(tx * ((cam.height + 15) // 16)):
        y, x = t // tx * 16, t % tx * 16
        ids = np.unique(sel[y:y + 16, x:x + 16])
        ids = ids[ids >= 0]
        lst = gids[offs[t]:offs[t + 1]]
        pos = np.flatnonzero(np.isin(lst, ids))
        res.append((ids.size, pos.max(initial=-1)))
    return np.array(res)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_scenes_reach_the_slot_paths(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _, _, _, n_small, corner = case
    distinct, position = _tiles(case).max(axis=0)
    assert distinct > (256 if n_small >= 900 and not corner else 32)
    if corner:
        assert position >= 8192
