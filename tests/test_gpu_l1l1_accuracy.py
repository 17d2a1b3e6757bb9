"""Rounding of the l1-l1 stage over its penalties (needs an MI355X): in FP32 its
distance from the FP64 oracle is that of the plain sweeps in FP32 arithmetic (the
Bregman variables summed from the differences h - x and D x, which are small
beside x), whatever the penalties are.  30 % above that is allowed for the segments
of the device's elimination; rounding a difference at the size of x doubles the
distance at a small mu1 / mu2.

Extreme ratios: as in the oracle, to 1e-5 (FP32) and 1e-10 (FP64)."""
import numpy as np
import pytest

from oracle import hyminor_oracle as HM

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_06979_amd import api
    return api


def _spectra(n, p, seed):
    rng = np.random.default_rng(seed)
    h = 0.5 + 0.03 * np.cumsum(rng.standard_normal((n, p)), axis=1)
    mask = rng.random((n, p)) < 0.02
    h[mask] += rng.choice([-1.0, 1.0], size=int(mask.sum()))
    return h.astype(np.float32)


def _fma(a, b, c):
    return (np.asarray(a, np.float64) * b + c).astype(np.float32)


def _plain_fp32(h, lam, mu1, mu2, iters):
    """Split Bregman sweeps in FP32 with one Thomas elimination per pixel."""
    f = np.float32
    n, p = h.shape
    d = np.full(p, mu1 + 2 * mu2)
    d[0] = d[-1] = mu1 + mu2
    beta = d.copy()
    for i in range(1, p):
        beta[i] = d[i] - mu2 * mu2 / beta[i - 1]
    inv, back = (1.0 / beta).astype(f), (mu2 / beta).astype(f)
    m1, m2, t1, t2 = f(mu1), f(mu2), f(1.0 / mu1), f(lam / mu2)
    x, b1, b2 = np.zeros((n, p), f), np.zeros((n, p), f), np.zeros((n, p - 1), f)
    for k in range(iters):
        a, c = h, np.zeros((n, p), f)
        if k:
            t = (h - x) + b1
            b1 = np.clip(t, -t1, t1)
            a = _fma(2, b1, h - t)
            v = (x[:, 1:] - x[:, :-1]) + b2
            b2 = np.clip(v, -t2, t2)
            c[:, :-1] = _fma(-2, b2, v)
        z, zp, cp = np.zeros((n, p), f), np.zeros(n, f), np.zeros(n, f)
        for i in range(p):
            zp = _fma(m2, zp, _fma(m1, a[:, i], m2 * (cp - c[:, i]))) * inv[i]
            cp = c[:, i]
            z[:, i] = zp
        for i in range(p - 2, -1, -1):
            z[:, i] = _fma(back[i], z[:, i + 1], z[:, i])
        x = z
    return x


@pytest.mark.parametrize("mu1,mu2", [(1.0, 1.0), (0.6, 1.3), (0.02, 1.0), (1.0, 0.01), (0.001, 1.0), (5.0, 3.0)])
@pytest.mark.parametrize("p", [40, 103, 144])
def test_fp32_rounding(p, mu1, mu2):
    api = _api()
    h = _spectra(1280, p, p)
    ref = HM.l1l1_split_bregman(h.astype(np.float64), 0.55, mu1, mu2, 50)
    plain = np.linalg.norm(_plain_fp32(h, 0.55, mu1, mu2, 50) - ref) / np.linalg.norm(ref)
    X = api.l1l1_spectral(torch.tensor(h.reshape(32, 40, p), device="cuda"), 0.55, mu1, mu2, 50)
    err = np.linalg.norm(X.cpu().numpy().reshape(-1, p) - ref) / np.linalg.norm(ref)
    print("l1l1 p", p, "mu", mu1, mu2, "device", err, "plain", plain, flush=True)
    assert err <= 1.3 * plain


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("mu1,mu2,scale", [(1.0, 1e-30, 1e9), (1e4, 1e-12, 1e25), (1e-4, 1e4, 1e-20)])
def test_extreme_ratios(dtype, mu1, mu2, scale):
    api = _api()
    h = (_spectra(80, 70, 3).astype(np.float64) * scale).astype(dtype)
    lam = 0.05 * scale
    ref = HM.l1l1_split_bregman(h.astype(np.float64), lam, mu1, mu2, 6)
    X = api.l1l1_spectral(torch.tensor(h.reshape(8, 10, 70), device="cuda"), lam, mu1, mu2, 6).cpu().numpy()
    err = np.linalg.norm((X.reshape(-1, 70) - ref) / scale) / np.linalg.norm(ref / scale)
    print("l1l1 extreme", dtype.__name__, mu1, mu2, scale, err, flush=True)
    assert err <= (1e-5 if dtype == np.float32 else 1e-10)
