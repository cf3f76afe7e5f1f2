"""Passes in row blocks that carry the previous block's transpose (FP32 above
4096; SCINT_SCREEN_JOBS sets the number of blocks): every block count gives the
one-block result bit for bit.  5000 has a ragged last band of 8 rows and blocks
that end inside a screen; the counts reach more blocks than screens, and a
single one."""
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


@pytest.mark.parametrize("N,n", [(5000, 1), (5000, 3), (8192, 1)])
def test_blocks_equal_one_block(S, monkeypatch, N, n):
    z = N / LAM  # conjugate planes, for the aperture mode too
    phi = torch.tensor(inputs.phase_field(256, 1)[0].astype(np.float32), device="cuda")
    phi = phi.repeat(1, -(-N // 256), -(-N // 256))[0][:N, :N].contiguous()[None]

    def outputs():
        a = S.ps_screen_fresnel(N, 1.0, 20.0, 11 / 3, 5, LAM, z, n_real=n)
        b = S.ps_screen_fresnel(N, 1.0, 20.0, 11 / 3, 5, LAM, z, n_real=n, want_phi=True, want_field=True)
        return (a,) + b + (S.fresnel_propagate(phi, 1.0, LAM, z), S.fresnel_aperture(phi, 1.0, LAM, z),
                           S.fresnel_propagate_field(phi, 1.0, LAM, z)[1])

    monkeypatch.setenv("SCINT_SCREEN_JOBS", "1")
    ref = outputs()
    assert all(abs(float(x.mean()) - 1.0) < 1e-3 for x in (ref[0], ref[1], ref[4]))
    for jobs in (2, 4, 7):
        monkeypatch.setenv("SCINT_SCREEN_JOBS", str(jobs))
        for x, y in zip(outputs(), ref):
            assert torch.equal(x, y), jobs
