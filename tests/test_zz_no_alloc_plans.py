"""fresnel_propagate_noalloc at the sizes whose FP64 plan is not FP32's (80, 200)
and at the other small plans: its device-built twiddle table is that of the plan
it runs, so the result lies within the bars of the parity tests of the oracle
(FP64 1e-10 of the mean; FP32 RMS 2e-5, max 1e-3)."""
import numpy as np
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu

LAM = 5e-7


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("N", [64, 80, 128, 200, 256, 400])
def test_noalloc_plans(oracle, N, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0514_amd import scint as S
    S.load_library()
    rho = N / 10.0
    z = 2 * np.pi * rho ** 2 / LAM
    phi = inputs.phase_field(N, N, sigma=1.5, n=3).astype(np.float64 if dtype == torch.float64 else np.float32)
    I = S.fresnel_propagate_noalloc(torch.tensor(phi, device="cuda"), 1.0, LAM, z, 0.8)
    torch.cuda.synchronize()
    for b in range(3):
        ref = oracle.propagate(phi[b].astype(np.float64), rho, 0.8)
        d = I[b].double().cpu().numpy() - ref
        rms, top = np.sqrt(np.mean(d * d)) / ref.mean(), np.abs(d).max() / ref.mean()
        assert (rms < 1e-10 and top < 1e-10) if dtype == torch.float64 else (rms < 2e-5 and top < 1e-3), (rms, top)
