"""FP64 cubes on the FP64 matrix cores: Gram, projection and back-projection at
the edges of their tiles (band counts around multiples of 16 and 32, ranks
around multiples of 4, pixel counts that leave partial steps, image rows shorter
than a step, strided cubes)."""
import numpy as np
import pytest

from oracle import hyres_oracle as O
from paper_2204_06979_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_06979_amd import api
    return api


@pytest.mark.parametrize("H,W,p", [(1, 7, 2), (3, 3, 3), (67, 1, 15), (5, 13, 16), (40, 3, 17), (9, 29, 32),
                                   (64, 65, 33), (31, 33, 100), (7, 41, 224)])
@pytest.mark.parametrize("strided", [False, True])
def test_gram_f64(H, W, p, strided):
    api = _api()
    print("gram_f64", H, W, p, strided, flush=True)
    rng = np.random.default_rng(1000 * H + p)
    full = rng.standard_normal((H, W + 2, p + 3))
    Y = full[:, 1:W + 1, 2:p + 2] if strided else np.ascontiguousarray(full[:, 1:W + 1, 2:p + 2])
    Yt = torch.tensor(full, device="cuda")[:, 1:W + 1, 2:p + 2] if strided else torch.tensor(Y, device="cuda")
    _, G, _ = api.estimate_noise(Yt, return_gram=True)
    Y2 = np.asarray(Y).reshape(-1, p)
    # a sum of n products in any order: n eps sum |y_a y_b|
    tol = H * W * np.finfo(np.float64).eps * (np.abs(Y2).T @ np.abs(Y2))
    assert (np.abs(G.cpu().numpy() - Y2.T @ Y2) <= tol).all()


@pytest.mark.parametrize("H,W,p,r", [(17, 16, 16, 1), (21, 20, 17, 4), (24, 43, 33, 5), (19, 23, 48, 16),
                                     (40, 41, 224, 9)])
@pytest.mark.parametrize("strided", [False, True])
def test_products_f64(H, W, p, r, strided):
    api = _api()
    print("products_f64", H, W, p, r, strided, flush=True)
    cube = synth.mixing_cube(H + p, H, W, p, r, 10.0, 2, dtype=np.float64, keep_clean=False)
    lam = np.linspace(0.2, 2.0, r)
    if strided:
        buf = torch.zeros(H, W + 1, p + 1, dtype=torch.float64, device="cuda")
        buf[:, :W, :p] = torch.tensor(cube.Y)
        Yt = buf[:, :W, :p]
    else:
        Yt = torch.tensor(cube.Y, device="cuda")
    X, _ = api.denoise(Yt, r, 2, lam=torch.tensor(lam))
    ref = O.hyres(cube.Y, r, 2, lam=lam)["X"]
    assert np.linalg.norm(X.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref)
