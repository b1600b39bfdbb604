"""Kernel launches of calls that should need no more: counted as the nodes of a
captured graph."""

import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20927_amd as qr
    return qr


def _launches(call):
    call()  # whatever the first call sets up
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    n = ctypes.c_size_t()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("n,dim", [(100, 333), (1, 4), (7, 16), (64, 512)])
def test_bfloat16_encoder_is_one_launch(qr, n, dim):
    f = torch.randn(n, dim, device="cuda")
    out = torch.empty(n, dim, dtype=torch.bfloat16, device="cuda")
    assert _launches(lambda: qr._lib.qr_quantize_features(f, qr._lib.QR_BF16, out)) == 1
    assert torch.equal(out, f.to(torch.bfloat16))
