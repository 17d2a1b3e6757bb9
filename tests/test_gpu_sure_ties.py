"""Threshold search of tied values (needs an MI355X): integers and other grids, whose
histogram bins hold one value many times over, from one block's components to those
refined by all of them.  Thresholds are values of the component, so they compare
exactly with the FP64 oracle's; the risk at them is a sum of N terms.

A million integers took one block 2.0 ms value by value; a tenth of a millisecond
is what the same number of different values takes."""
import numpy as np
import pytest

from oracle import hyres_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [(3000, np.float32), (65536, np.float64), (70000, np.float32), (200001, np.float64), (1000003, np.float32),
         (1000003, np.float64), (3000000, np.float32), (2100000, np.float64), ((1 << 24) + 5, np.float32)]


def _api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_06979_amd import api
    return api


def _grid(N, step, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "mixture":
        x = rng.standard_normal(N)
        x[rng.random(N) < 0.05] *= 10
    elif kind == "laplace":
        x = rng.laplace(size=N) * 1.2
    else:                      # every hundredth value off the grid
        x = rng.standard_normal(N)
        x[rng.random(N) < 0.05] *= 10
        keep = rng.random(N) < 0.01
        y = np.round(x / step) * step
        y[keep] = x[keep]
        return y
    return np.round(x / step) * step


@pytest.mark.parametrize("N,dtype", SIZES)
@pytest.mark.parametrize("step", [1.0, 0.125, 1.0 / 64, 1.0 / 1024])
def test_ties(N, dtype, step):
    api = _api()
    kinds = ["mixture", "laplace", "some"] if N < 2000000 else ["mixture"]
    x = np.stack([_grid(N, step, k, N % 1000 + i) for i, k in enumerate(kinds)]).astype(dtype)
    lam, sure, st = api.sure_threshold(torch.tensor(x, device="cuda"))
    for i, k in enumerate(kinds):
        t, s = O.sure_threshold(x[i].astype(np.float64))
        print("ties", N, dtype.__name__, step, k, float(lam[i]), t, float(sure[i]), s, int(st[0]), flush=True)
        assert float(lam[i]) == t
        np.testing.assert_allclose(float(sure[i]), s, rtol=1e-10, atol=1e-10 * N)
    assert int(st[0]) == 0


@pytest.mark.parametrize("N,bound", [(1000003, 0.7), ((1 << 24) + 5, 2.0)])
def test_integers_time(N, bound):
    api = _api()
    x = torch.tensor(_grid(N, 1.0, "mixture", 1).astype(np.float32)[None], device="cuda")
    ts = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            api.sure_threshold(x)
        b.record()
        torch.cuda.synchronize()
        ts.append(a.elapsed_time(b) / 5)
    print("integers", N, "ms", min(ts), flush=True)
    assert min(ts) < bound
