"""Passes that store their fields by columns at 2000 to 4096, in both precisions,
against the FP64 oracle: screen + pattern, propagation, kept field, both forms
of the adjoint, aperture, smear, co-addition.  2000, 2560 and 4000 take fewer
rows per workgroup in their heavier passes; 4096 has three FP32 plans.

Tolerances: the bars of the parity tests (FP64 1e-10 of the mean; FP32 RMS
2e-5, max 1e-3; gradients rel L2 2e-5).
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


CASES = [(N, d, 0) for N in (2000, 2560, 4000, 4096) for d in (torch.float32, torch.float64)]
CASES += [(2048, torch.float32, 1), (4096, torch.float32, 1), (4096, torch.float32, 2), (2048, torch.float64, 0)]


@pytest.mark.parametrize("N,dtype,plan", CASES)
def test_column_passes_vs_oracle(S, oracle, monkeypatch, N, dtype, plan):
    rho, s, R, beta, seed = N / 12.0, 0.8, N / 100.0, 11 / 3, 23
    z = 2 * np.pi * rho ** 2 / LAM
    npdt = np.float64 if dtype == torch.float64 else np.float32
    phi = inputs.phase_field(N, N, sigma=1.5).astype(npdt)
    gI = np.random.default_rng(N).standard_normal((1, N, N)).astype(npdt)
    p64, g64 = phi[0].astype(np.float64), gI[0].astype(np.float64)
    t, g = torch.tensor(phi, device="cuda"), torch.tensor(gI, device="cuda")
    if dtype == torch.float32 and S.num_plan_variants(N) > 1:
        S.set_plan_variant(N, plan)
    try:
        I = S.fresnel_propagate(t, 1.0, LAM, z, s)
        If, field = S.fresnel_propagate_field(t, 1.0, LAM, z, s)
        grads = [S.fresnel_propagate_vjp(t, 1.0, LAM, z, g, s, field=field),
                 S.fresnel_propagate_vjp(t, 1.0, LAM, z, g, s)]
        Isf = S.ps_screen_fresnel(N, 1.0, R, beta, seed, LAM, z, dtype=dtype)
        Isp, phis = S.ps_screen_fresnel(N, 1.0, R, beta, seed, LAM, z, dtype=dtype, want_phi=True)
        lams = [0.9 * LAM, LAM, 1.15 * LAM]
        poly = S.illumination_polychromatic(t, 1.0, z, LAM, lams)
        ext = S.source_smear(I, 1.0, [N / 50.0])
        za = 1.2 * N / LAM
        ap = S.fresnel_aperture(t, 1.0, LAM, za)
    finally:
        if dtype == torch.float32 and S.num_plan_variants(N) > 1:
            S.set_plan_variant(N, -1)
    ref = oracle.propagate(p64, rho, s)
    close(I[0], ref, dtype)
    close(If[0], ref, dtype)
    gref = oracle.propagate_vjp(p64, rho, s, g64)
    for x in grads:
        close(x[0], gref, dtype)
    sref = oracle.screen(N, R, beta, seed, 0)
    close(phis[0], sref, dtype)
    pref = oracle.propagate(sref, rho)
    close(Isf[0], pref, dtype)
    close(Isp[0], pref, dtype)
    close(poly[0], oracle.polychromatic(p64, 1.0, z, LAM, lams), dtype)
    close(ext[0, 0], oracle.smear(I[0].double().cpu().numpy(), N / 50.0), dtype)
    close(ap[0], oracle.fresnel_aperture(p64, oracle.fresnel_radius_px(1.0, LAM, za), 1.0, 10.0), dtype)
