"""Smear of an odd number of patterns, the last one a pair whose second is zero,
with all radii inverted in one launch: equal bit for bit to every pattern
smeared on its own pair, and within the bars of the oracle (FP64 1e-10, FP32
RMS 2e-5 and max 1e-3 of the mean)."""
import numpy as np
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0514_amd import scint
    scint.load_library()
    return scint


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("N,n,n_r", [(16, 3, 1), (100, 5, 2), (256, 3, 3), (640, 1, 5), (1280, 3, 2), (5000, 3, 2)])
def test_odd_batches(S, oracle, N, n, n_r, dtype):
    if N == 5000 and dtype == torch.float64:
        pytest.skip("one large size is enough")
    radii = [1.5 + 3.0 * r for r in range(n_r)]
    I = torch.tensor(inputs.intensity_field(N, N, n=n), dtype=dtype, device="cuda")
    out = S.source_smear(I, 1.0, radii)
    assert out.shape == (n, n_r, N, N)
    alone = S.source_smear(I[n - 1:].contiguous(), 1.0, radii)
    assert torch.equal(out[n - 1], alone[0])
    for q in range(n // 2):
        assert torch.equal(out[2 * q:2 * q + 2], S.source_smear(I[2 * q:2 * q + 2].contiguous(), 1.0, radii))
    for b in {0, n - 1}:
        i64 = I[b].double().cpu().numpy()
        for r, R in enumerate(radii[:2]):
            d = out[b, r].double().cpu().numpy() - oracle.smear(i64, R)
            rms, top = np.sqrt(np.mean(d * d)) / i64.mean(), np.abs(d).max() / i64.mean()
            assert (rms < 1e-10 and top < 1e-10) if dtype == torch.float64 else (rms < 2e-5 and top < 1e-3)
