"""Co-addition over batches whose fields exceed the cache: the first pass takes
more rows per workgroup there (up to 320), with the same arithmetic, so a
screen's pattern equals that of a small batch bit for bit; the kept field and
the recomputing adjoint, which run the same pass once, too.  Batches end inside
a row group."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LAM = 5e-7


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0514_amd import scint
    scint.load_library()
    return scint


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("N", [64, 80, 128, 160, 256, 320])
def test_large_batch_equals_small(S, N, dtype):
    z = 2 * np.pi * (N / 10.0) ** 2 / LAM
    lams = [LAM * (0.8 + 0.05 * j) for j in range(8)]
    eb = 8 if dtype == torch.float32 else 16
    n = (256 << 20) // (8 * N * N * eb) + 3  # just above 256 MiB with eight wavelengths
    g = torch.Generator(device="cuda").manual_seed(N)
    phi = torch.randn((n, N, N), dtype=dtype, device="cuda", generator=g)
    I = S.illumination_polychromatic(phi, 1.0, z, LAM, lams)
    for b in (0, n // 2, n - 3):
        assert torch.equal(I[b:b + 3], S.illumination_polychromatic(phi[b:b + 3].contiguous(), 1.0, z, LAM, lams))
    assert float(I.mean()) == pytest.approx(1.0, abs=1e-4)
    n = (256 << 20) // (N * N * eb) + 3  # one field
    phi = torch.randn((n, N, N), dtype=dtype, device="cuda", generator=g)
    w = torch.rand((n, N, N), dtype=dtype, device="cuda", generator=g)
    If, field = S.fresnel_propagate_field(phi, 1.0, LAM, z)
    grad = S.fresnel_propagate_vjp(phi, 1.0, LAM, z, w)
    for b in (0, n - 3):
        p, v = phi[b:b + 3].contiguous(), w[b:b + 3].contiguous()
        i, f = S.fresnel_propagate_field(p, 1.0, LAM, z)
        assert torch.equal(If[b:b + 3], i) and torch.equal(field[b:b + 3], f)
        assert torch.equal(grad[b:b + 3], S.fresnel_propagate_vjp(p, 1.0, LAM, z, v))
