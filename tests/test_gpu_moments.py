"""Mean and modulation index in one read of the region
(ps_modulation_index, ps_modulation_index_region) against numpy in FP64: one
pixel, single rows and columns, odd offsets (no 16-byte loads), full width;
patterns whose mean is far from zero, and with an infinity or a NaN.

Tolerance: the reference's own two-pass sums round at N 2^-53 (1e-12 for the
largest region here); a mean 1e4 standard deviations from zero costs a factor
1e4 in m, so rel 1e-8 there and 1e-11 elsewhere."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

REGIONS = [(0, 0, 100, 100), (3, 5, 1, 1), (0, 7, 100, 1), (1, 0, 1, 100), (1, 1, 97, 51), (0, 2, 100, 64), (4, 0, 64, 3)]


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0514_amd import scint
    scint.load_library()
    return scint


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("offset", [0.0, 1e4])
@pytest.mark.parametrize("N,n", [(100, 3), (1000, 2)])
def test_moments(S, dtype, offset, N, n):
    I = torch.tensor(offset + np.random.default_rng(N).exponential(1.0, (n, N, N)), dtype=dtype, device="cuda")
    h = I.double().cpu().numpy()
    rel = 1e-8 if offset else 1e-11
    m, mean = S.ps_modulation_index(I, want_mean=True)
    assert mean == pytest.approx(list(h.mean((1, 2))), rel=1e-12)
    assert m == pytest.approx(list(h.std((1, 2)) / h.mean((1, 2))), rel=rel)
    for x0, y0, w, hh in REGIONS + [(11, 13, N - 30, N - 17)]:
        r = h[:, y0:y0 + hh, x0:x0 + w]
        m, mean = S.ps_modulation_index_region(I, x0, y0, w, hh, want_mean=True)
        assert mean == pytest.approx(list(r.mean((1, 2))), rel=1e-12), (x0, y0, w, hh)
        assert m == pytest.approx(list(r.std((1, 2)) / r.mean((1, 2))), rel=rel, abs=1e-15), (x0, y0, w, hh)


@pytest.mark.parametrize("at", [(0, 0), (57, 3), (99, 99)])
@pytest.mark.parametrize("value", [math.inf, math.nan])
def test_moments_of_unbounded_patterns(S, at, value):
    I = torch.rand((2, 100, 100), device="cuda") + 0.5
    good = S.ps_modulation_index(I[1:].contiguous())
    I[0][at] = value
    m, mean = S.ps_modulation_index(I, want_mean=True)
    assert math.isnan(m[0]) and (mean[0] == value or math.isnan(value) and math.isnan(mean[0]))
    assert m[1] == good[0]
