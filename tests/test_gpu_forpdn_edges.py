"""FORPDN at the edges of its kernels (needs an MI355X): band counts around the
16-band chunks of the tridiagonal solve and with and without 16-byte rows,
levels down to one position, widths of one and several 32-position strips, and
rows that are not 16-byte aligned.  Noise and thresholds are given, so that the
output is compared with the oracle alone: relative Frobenius 1e-10 (FP64) and
1e-5 (FP32), as for the other FORPDN cases."""
import numpy as np
import pytest

from oracle import forpdn_oracle as F

import parity_metrics as PM

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(4, 4, 2, 1), (5, 7, 3, 1), (9, 70, 15, 2), (7, 131, 16, 2), (17, 66, 17, 3), (16, 64, 32, 3),
          (7, 33, 36, 2), (12, 13, 145, 2), (11, 19, 208, 2), (10, 21, 209, 2), (7, 40, 224, 2)]


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("pad", [0, 1, 4])
def test_forpdn_edges(shape, dtype, pad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_06979_amd import api
    H, W, p, L = shape
    rng = np.random.default_rng(H * 1000 + W + p)
    Y = rng.random((H, W, p)).astype(dtype)
    sig = 0.02 + 0.05 * rng.random(p)
    lam = np.array([300.0, 7.0, 0.3, 0.01])[:L + 1]
    buf = torch.zeros(H, W, p + pad, dtype=torch.tensor(Y).dtype, device="cuda")
    buf[:, :, :p] = torch.tensor(Y, device="cuda")
    out = torch.full_like(buf, 7.0)
    api.forpdn(buf[:, :, :p], L, sigma=torch.tensor(sig), lam=torch.tensor(lam), X=out[:, :, :p])
    ref = F.forpdn(Y.astype(np.float64), L, sigma=sig, lam=lam)
    PM.assert_close(out[:, :, :p].cpu().numpy(), ref["X"], 1e-10 if dtype == np.float64 else 1e-5, str(shape))
    assert bool((out[:, :, p:] == 7.0).all())
