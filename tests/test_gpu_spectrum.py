"""Every eigenvalue of the whitened Gram (needs an MI355X), not only the leading
ones: band counts of each remainder modulo four, at both sides of the edges of
the small solve's layouts, against the FP64 oracle.  With all eigenvalues asked
for, four of them share the sixteen lanes that hold the tridiagonal matrix, so
the last of them run beside lanes that have none.

Tolerance: an eigenvalue is good to 224 eps of the largest (5e-14); 1e-11 of it
is allowed, a thousandth of the smallest eigenvalue here and less."""
import numpy as np
import pytest

from oracle import hyres_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BANDS = [5, 31, 33, 34, 35, 47, 49, 63, 65, 66, 67, 95, 97, 103, 127, 129, 130, 143, 145, 159, 161, 175, 177, 191, 193,
         207, 209, 222, 223, 224]


def _cube(p, r):
    rng = np.random.default_rng(p)
    sig = 0.5 + rng.random(p)
    Q, _ = np.linalg.qr(rng.standard_normal((p, r)))
    A = rng.standard_normal((30 * 40, r)) * (30.0 / 1.7 ** np.arange(r))
    return ((A @ Q.T + rng.standard_normal((30 * 40, p))) * sig).reshape(30, 40, p)


@pytest.mark.parametrize("p", BANDS)
def test_all_eigenvalues(p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_06979_amd import api
    r = 2 if p < 8 else 5
    Y = _cube(p, r)
    Yd = torch.tensor(Y, device="cuda")
    ref = O.hyres(Y, r, 2)
    w = ref["evals"]
    ev = api.subspace(Yd, r, sigma=torch.tensor(ref["sigma"], device="cuda"))[1].cpu().numpy()
    print("spectrum p", p, np.max(np.abs(ev - w)) / w[0], flush=True)
    np.testing.assert_allclose(ev, w, rtol=1e-11, atol=1e-11 * w[0])
    # ... through a whole solve, its noise estimated (a few 1e-9 of sigma: 1e-8 of an eigenvalue)
    info = api.denoise(Yd, r, 2, all_evals=True)[1]
    np.testing.assert_allclose(info["evals"].cpu().numpy(), w, rtol=2e-8)
    # the rank by SURE sums over all of them
    info = api.denoise(Yd, r, 2, rank_rule="sure")[1]
    np.testing.assert_allclose(info["evals"].cpu().numpy(), w, rtol=2e-8)
    assert int(info["rank"].cpu()[0]) == O.hyres(Y, r, 2, rank_rule="sure")["rank"]
