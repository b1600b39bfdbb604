"""Both backward passes at the widths where their waves share the columns
differently (dense: 128 a wave; Q-Render: 32-column blocks over four or eight
waves, some of which take other pixels instead), on a picture with ragged edges,
against the FP64 oracle under test_gpu_backward's element-wise bound."""

import pytest
import torch

import synth
from tests.test_gpu_backward import _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20927_amd as qr
    return qr


@pytest.mark.parametrize("dim", [16, 112, 128, 144, 240, 256, 272, 384, 400, 496])
@pytest.mark.parametrize("K,storage", [(8, "bf16"), (24, "f32")])
def test_widths(qr, dim, K, storage):
    sc = synth.make_tiny(dim, n=500, dim=dim)
    cam = synth.tiny_camera(38)
    cam.height, cam.cy = 21, 10.5
    _run(qr, sc, cam, K, storage=storage, seed=K)
