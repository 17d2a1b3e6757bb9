"""The small solve on Gram matrices of any scale (needs an MI355X): a cube times a
power of two has the same eigenvectors and the eigenvalues times its square, down
to squares of the tridiagonalisation next to the smallest normal number.

Tolerances: against the FP64 oracle, 1e-11 of an eigenvalue (224 eps of the largest,
5e-14, over a smallest eigenvalue a two-hundredth of it) and 1e-9 on V, as for a
cube of ordinary scale."""
import numpy as np
import pytest

from oracle import hyres_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [7, 33, 103, 224])
@pytest.mark.parametrize("e", [-240, -183, 0, 240])
def test_subspace_scale(p, e):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_06979_amd import api
    r = 2 if p < 8 else 5
    rng = np.random.default_rng(p)
    Q, _ = np.linalg.qr(rng.standard_normal((p, r)))
    A = rng.standard_normal((30 * 40, r)) * (10.0 / 1.7 ** np.arange(r))
    Y = (A @ Q.T + rng.standard_normal((30 * 40, p))).reshape(30, 40, p)
    V_ref, w_ref = O.subspace(Y.reshape(-1, p), r)
    V, ev, st = [t.cpu().numpy() for t in api.subspace(torch.tensor(np.ldexp(Y, e), device="cuda"), r)]
    ev = np.ldexp(ev, -2 * e)
    print("scale p", p, "2^%d" % e, np.max(np.abs(ev / w_ref - 1)), np.max(np.abs(V - V_ref)), flush=True)
    assert st[0] == 0
    np.testing.assert_allclose(ev, w_ref, rtol=1e-11)
    np.testing.assert_allclose(V, V_ref, atol=1e-9)
