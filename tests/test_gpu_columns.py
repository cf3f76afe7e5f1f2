"""Passes that store their field by columns (up to 4096; real arrays up to
1024): every entry point that goes through them, on batches whose rows do not
fill whole workgroups, against the FP64 oracle.  Sizes on both sides of each
rule: one row group only (16), rows of a few lanes (40, 100), the last size
with real arrays by columns (1024) and the first without (1280).

Tolerances: the bars of the parity tests (FP64 to rounding, 1e-10 of the
mean; FP32 RMS 2e-5, max 1e-3 of the mean; gradients rel L2 2e-5).
"""
import numpy as np
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu

LAM = 5e-7


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0514_amd import scint
    scint.load_library()
    return scint


def close(a, ref, dtype):
    d = a.detach().double().cpu().numpy() - ref
    scale = np.sqrt(np.mean(ref * ref))
    rms, top = np.sqrt(np.mean(d * d)) / scale, np.abs(d).max() / np.abs(ref).max()
    bars = (1e-10, 1e-10) if dtype == torch.float64 else (2e-5, 1e-3)
    assert rms < bars[0] and top < bars[1], (rms, top)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("N,n", [(16, 1), (16, 5), (40, 3), (100, 3), (1024, 1), (1280, 1)])
def test_column_passes_vs_oracle(S, oracle, N, n, dtype):
    rho, s, R, beta, seed = N / 10.0, 0.8, max(2.5, N / 100.0), 11 / 3, 11
    z = 2 * np.pi * rho ** 2 / LAM
    npdt = np.float64 if dtype == torch.float64 else np.float32
    phi = inputs.phase_field(N, N + n, sigma=1.5, n=n).astype(npdt)
    gI = np.random.default_rng(N).standard_normal((n, N, N)).astype(npdt)
    t, g = torch.tensor(phi, device="cuda"), torch.tensor(gI, device="cuda")
    I = S.fresnel_propagate(t, 1.0, LAM, z, s)
    If, field = S.fresnel_propagate_field(t, 1.0, LAM, z, s)
    grad = S.fresnel_propagate_vjp(t, 1.0, LAM, z, g, s, field=field)
    grad_again = S.fresnel_propagate_vjp(t, 1.0, LAM, z, g, s)
    Isf = S.ps_screen_fresnel(N, 1.0, R, beta, seed, LAM, z, n_real=n, dtype=dtype)
    Isp, phis = S.ps_screen_fresnel(N, 1.0, R, beta, seed, LAM, z, n_real=n, dtype=dtype, want_phi=True)
    ext = S.source_smear(I, 1.0, [2.0, N / 12.0])
    for b in {0, n - 1}:
        p64, g64 = phi[b].astype(np.float64), gI[b].astype(np.float64)
        ref = oracle.propagate(p64, rho, s)
        close(I[b], ref, dtype)
        close(If[b], ref, dtype)
        gref = oracle.propagate_vjp(p64, rho, s, g64)
        close(grad[b], gref, dtype)
        close(grad_again[b], gref, dtype)
        sref = oracle.screen(N, R, beta, seed, b)
        close(phis[b], sref, dtype)
        pref = oracle.propagate(sref, rho)
        close(Isf[b], pref, dtype)
        close(Isp[b], pref, dtype)
        i64 = I[b].double().cpu().numpy()
        for k, r in enumerate((2.0, N / 12.0)):
            close(ext[b, k], oracle.smear(i64, r), dtype)


@pytest.mark.parametrize("N,n,m", [(64, 1, 9), (100, 3, 5), (1280, 1, 3)])
def test_split_wavelengths_equal_unsplit(S, monkeypatch, N, n, m):
    # several workgroups per row group, each with a part of the wavelengths
    phi = torch.tensor(inputs.phase_field(N, 3, n=n).astype(np.float32), device="cuda")
    z = 2 * np.pi * (N / 10.0) ** 2 / LAM
    lams = [LAM * (0.9 + 0.03 * j) for j in range(m)]
    a = S.illumination_polychromatic(phi, 1.0, z, LAM, lams)
    monkeypatch.setenv("SCINT_ITER_SPLIT", "1")
    b = S.illumination_polychromatic(phi, 1.0, z, LAM, lams)
    assert torch.equal(a, b)
