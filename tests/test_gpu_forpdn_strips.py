"""FORPDN of wide images (needs an MI355X): several strips of 32 blocks of the
analysis (64 outputs each) and of 32 positions of the synthesis, the last one ragged
or whole, with one band and with 16 bytes of bands per thread.  Noise and thresholds
are given; relative Frobenius 1e-10 (FP64) and 1e-5 (FP32) against the oracle, as
for the other FORPDN cases."""
import numpy as np
import pytest

from oracle import forpdn_oracle as F

import parity_metrics as PM

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape", [(5, 259, 3, 1), (7, 256, 16, 2), (9, 515, 3, 2), (5, 515, 16, 1), (33, 1027, 4, 3)])
@pytest.mark.parametrize("pad", [0, 1])
def test_forpdn_strips(shape, dtype, pad):
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
