"""FFT plans of 64 to 256 with few elements per thread.

Rounding: FP32 propagation against FP64 of the same phases, RMS over 24 seeds
of two screens, may not exceed what the plans with 16 and 20 elements per
thread gave on the same inputs ({8,8}, {4,20}, {16,8}, {20,10}, {16,16}: the
bounds below, measured with them).

80, 128 and 200 against the oracle through every entry point that runs the
plans, on batches, with the bars of the parity tests (FP64 1e-10 of the mean;
FP32 RMS 2e-5, max 1e-3; gradients rel L2 2e-5).
"""
import math

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


@pytest.mark.parametrize("N,bound", [(64, 4.0570e-07), (80, 2.3433e-07), (128, 4.6634e-07), (200, 3.9902e-07),
                                     (256, 4.7703e-07)])
def test_fp32_rounding(S, N, bound):
    errors = []
    for seed in range(24):
        g = torch.Generator().manual_seed(1000 * N + seed)
        phi = torch.randn(2, N, N, generator=g, dtype=torch.float32) * 2
        z = 2 * math.pi * 8.0 ** 2
        a = S.fresnel_propagate(phi.cuda(), 1.0, 1.0, z).double()
        b = S.fresnel_propagate(phi.double().cuda(), 1.0, 1.0, z)
        errors.append(float((a - b).pow(2).mean().sqrt() / b.pow(2).mean().sqrt()))
    mean = sum(errors) / len(errors)
    print("N=%d rms error %.4e, bound %.4e" % (N, mean, bound))
    assert mean <= bound


def close(a, ref, dtype):
    d = a.detach().double().cpu().numpy() - ref
    scale = np.sqrt(np.mean(ref * ref))
    rms, top = np.sqrt(np.mean(d * d)) / scale, np.abs(d).max() / np.abs(ref).max()
    bars = (1e-10, 1e-10) if dtype == torch.float64 else (2e-5, 1e-3)
    assert rms < bars[0] and top < bars[1], (rms, top)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("N,n", [(80, 1), (80, 7), (128, 1), (128, 5), (200, 1), (200, 3)])
def test_small_plans_vs_oracle(S, oracle, N, n, dtype):
    rho, s, R, beta, seed = N / 10.0, 0.8, max(2.5, N / 100.0), 11 / 3, 17
    z = 2 * np.pi * rho ** 2 / LAM
    npdt = np.float64 if dtype == torch.float64 else np.float32
    phi = inputs.phase_field(N, N + n, sigma=1.5, n=n).astype(npdt)
    gI = np.random.default_rng(N).standard_normal((n, N, N)).astype(npdt)
    t, g = torch.tensor(phi, device="cuda"), torch.tensor(gI, device="cuda")
    lams, w = [0.8 * LAM, 0.9 * LAM, LAM, 1.2 * LAM], [0.5, 1.0, 2.0, 0.7]
    I = S.fresnel_propagate(t, 1.0, LAM, z, s)
    If, field = S.fresnel_propagate_field(t, 1.0, LAM, z, s)
    grad = S.fresnel_propagate_vjp(t, 1.0, LAM, z, g, s, field=field)
    grad_again = S.fresnel_propagate_vjp(t, 1.0, LAM, z, g, s)
    poly = S.illumination_polychromatic(t, 1.0, z, LAM, lams, w)
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
        close(poly[b], oracle.polychromatic(p64, 1.0, z, LAM, lams, w), dtype)
        sref = oracle.screen(N, R, beta, seed, b)
        close(phis[b], sref, dtype)
        pref = oracle.propagate(sref, rho)
        close(Isf[b], pref, dtype)
        close(Isp[b], pref, dtype)
        i64 = I[b].double().cpu().numpy()
        for k, r in enumerate((2.0, N / 12.0)):
            close(ext[b, k], oracle.smear(i64, r), dtype)
