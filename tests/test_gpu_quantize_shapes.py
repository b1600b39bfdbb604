"""The storage encoders at the widths, row counts and alignments where their
kernels differ, bit for bit against the oracle's encoders; rows of zeros,
e4m3 subnormals, ties and the largest magnitudes among them."""

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20927_amd as qr
    return qr


def _table(n, dim):
    rng = np.random.default_rng(n * 1000 + dim)
    f = rng.standard_normal((n, dim)).astype(np.float32)
    f *= np.exp2(rng.integers(-14, 3, (n, dim))).astype(np.float32)  # down to the subnormals of the codes
    f[0, :] = 0.0
    if n > 1:  # scale 1: codes of the values themselves, ties to even among them
        f[1, :] = (rng.integers(-1792, 1793, dim) / 4.0).astype(np.float32)
        f[1, 0] = 448.0
    return f


@pytest.mark.parametrize("n,dim,skip", [(1, 4, 0), (7, 12, 0), (130, 16, 0), (9, 100, 0), (33, 256, 0), (17, 260, 0),
                                        (8, 512, 0), (5, 516, 0), (3, 1024, 0), (3, 1028, 0), (6, 333, 0), (6, 64, 1)])
def test_encoders(qr, n, dim, skip):
    f = _table(n, dim)
    store = torch.zeros(n * dim + skip, device="cuda")  # skip: a table that starts off the 16-byte boundary
    t = store[skip:].view(n, dim)
    t.copy_(torch.from_numpy(f))
    codes, scale = qr.quantize(t, "fp8")
    want, ws = oracle.quant.e4m3_quantize(f)
    assert np.array_equal(scale.cpu().numpy(), np.asarray(ws, np.float32))
    assert np.array_equal(codes.cpu().numpy(), want)
    b, _ = qr.quantize(t, "bf16")
    assert np.array_equal(b.view(torch.int16).cpu().numpy().view(np.uint16), oracle.quant.bf16_encode(f))
