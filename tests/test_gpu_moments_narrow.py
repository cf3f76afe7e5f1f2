"""ps_modulation_index_region on narrow regions, whose threads keep to one
column each: widths on both sides of every power of two up to 256 and just past
it, few and many rows, at odd offsets, against numpy in FP64 (mean rel 1e-12, m
rel 1e-11: a few thousand rounded sums); and a strip of two columns may not cost
more than the whole pattern does (read by whole rows it took eight times that).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0514_amd import scint
    scint.load_library()
    return scint


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("w", [1, 2, 3, 5, 64, 65, 128, 129, 255, 256, 257])
def test_widths(S, dtype, w):
    N, n = 1000, 2
    I = torch.tensor(np.random.default_rng(w).exponential(1.0, (n, N, N)), dtype=dtype, device="cuda")
    host = I.double().cpu().numpy()
    for x0, y0, h in ((0, 0, N), (N - w, 3, 1), (5, 1, 2), (7, 11, 4 * 256 + 1 - 300), (1, 0, N - 1)):
        r = host[:, y0:y0 + h, x0:x0 + w]
        m, mean = S.ps_modulation_index_region(I, x0, y0, w, h, want_mean=True)
        assert mean == pytest.approx(list(r.mean((1, 2))), rel=1e-12), (x0, y0, h)
        assert m == pytest.approx(list(r.std((1, 2)) / r.mean((1, 2))), rel=1e-11, abs=1e-15), (x0, y0, h)


def test_strip_costs_no_more_than_the_pattern(S):
    N = 2048
    I = torch.rand((2, N, N), device="cuda") + 0.5

    def best(f):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        f()
        t = []
        for _ in range(10):
            a.record()
            f()
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    whole, strip = best(lambda: S.ps_modulation_index(I)), best(lambda: S.ps_modulation_index_region(I, 5, 0, 2, N))
    print("whole %.4f ms, strip %.4f ms" % (whole, strip))
    assert strip < 3 * whole


def test_squares_that_overflow(S):
    # the deviations are finite and their squares are not: m is infinite, as numpy's std is
    I = 1e200 * (torch.rand((2, 100, 100), dtype=torch.float64, device="cuda") + 0.5)
    I[1] *= 1e-200
    for m, mean in (S.ps_modulation_index(I, want_mean=True), S.ps_modulation_index_region(I, 3, 5, 90, 80, True)):
        assert m[0] == float("inf") and 0.9e200 < mean[0] < 1.1e200
        assert m[1] == pytest.approx(0.29, abs=0.02)
