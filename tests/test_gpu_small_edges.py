"""The small solve and the l1-l1 stage at the edges of their layouts (needs an
MI355X): every multiple of 16 bands and its neighbours (columns per lane, waves
and rows in LDS change there), and band counts around the segment lengths of
the l1-l1 elimination, against the FP64 oracle.

Tolerances: the Gram matrices here have a condition below 1e5, so sigma is good
to 224 eps 1e5 = 5e-9; the eigenvalues to 224 eps of the largest (5e-14, 1e-11
allowed); V to eps of the largest eigenvalue over the smallest gap, below 1e4,
so to 1e-9.  l1-l1: 1e-10 in FP64 and 1e-5 in FP32, as in its other cases."""
import numpy as np
import pytest

from oracle import hyminor_oracle as HM
from oracle import hyres_oracle as O

import parity_metrics as PM

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BANDS = [3] + sorted({b for m in range(16, 225, 16) for b in (m - 1, m, m + 1) if b <= 224})


def _api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_06979_amd import api
    return api


@pytest.mark.parametrize("p", BANDS)
def test_small_solve_edges(p):
    api = _api()
    H, W = 30, 40
    r = 2 if p < 8 else 5
    rng = np.random.default_rng(p)
    sig = 0.5 + rng.random(p)
    # components of well separated strength over band-scaled noise
    Q, _ = np.linalg.qr(rng.standard_normal((p, r)))
    A = rng.standard_normal((H * W, r)) * (30.0 / 1.7 ** np.arange(r))
    Y = ((A @ Q.T + rng.standard_normal((H * W, p))) * sig).reshape(H, W, p)
    s_dev = api.estimate_noise(torch.tensor(Y, device="cuda"))[0].cpu().numpy()
    s_ref = O.noise_estimate(Y.reshape(-1, p))
    print("small p", p, "sigma", np.max(np.abs(s_dev / s_ref - 1)), flush=True)
    np.testing.assert_allclose(s_dev, s_ref, rtol=5e-9)
    V, ev = [t.cpu().numpy() for t in api.subspace(torch.tensor(Y, device="cuda"), r, sigma=torch.tensor(s_ref, device="cuda"))[:2]]
    V_ref, w_ref = O.subspace(Y.reshape(-1, p) / s_ref, r)
    print("   evals", np.max(np.abs(ev[:r] / w_ref[:r] - 1)), "V", np.max(np.abs(V - V_ref)), flush=True)
    np.testing.assert_allclose(ev[:r], w_ref[:r], rtol=1e-11)
    np.testing.assert_allclose(V, V_ref, atol=1e-9)


@pytest.mark.parametrize("dtype,p", [(np.float32, p) for p in (33, 36, 63, 72, 73, 136, 137, 145, 160, 192, 193, 208, 209)]
                         + [(np.float64, p) for p in (31, 48, 49, 64, 65, 112, 128, 129, 192, 193)])
def test_l1l1_segment_edges(dtype, p):
    api = _api()
    H, W = 7, 19
    rng = np.random.default_rng(p)
    h = 1.0 + 0.1 * np.cumsum(rng.standard_normal((H, W, p)), axis=2)
    mask = rng.random((H, W, p)) < 0.03
    h[mask] += rng.choice([-1.5, 2.0], size=int(mask.sum()))
    h = h.astype(dtype)
    X = api.l1l1_spectral(torch.tensor(h, device="cuda"), 0.9, 0.6, 1.3, 25).cpu().numpy()
    ref = HM.l1l1_split_bregman(h.astype(np.float64), 0.9, 0.6, 1.3, 25)
    PM.assert_close(X, ref, 1e-10 if dtype == np.float64 else 1e-5, "l1l1 p=%d" % p)
