"""FORPDN of band counts without 16-byte rows (needs an MI355X): a band fewer costs
little more than the full count.  191 and 192 bands of FP32 take 295 and 263 us for
256 x 256 pixels (398 and 274 with the rows' addresses spilled)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_odd_band_count_time():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_06979_amd import api

    def ms(p):
        g = torch.Generator(device="cuda")
        g.manual_seed(p)
        Y = torch.rand(256, 256, p, generator=g, device="cuda")
        X = torch.empty_like(Y)
        sig = torch.full((p,), 0.1, dtype=torch.float64, device="cuda")
        ts = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                api.forpdn(Y, 4, sigma=sig, X=X)
            b.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(b) / 20)
        return min(ts[1:])

    odd, full = ms(191), ms(192)
    print("forpdn 191", odd, "192", full, flush=True)
    assert odd < 1.28 * full
