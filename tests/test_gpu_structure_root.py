"""R_diff^rec by several levels of bisection per launch, and D at one radius
per workgroup (ps_structure_function): the root where it lies near either end
of its range, where it is not bracketed, and more radii than one launch takes,
against the FP64 oracle (rel 1e-9, the bar of the FP64 structure tests)."""
import math

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


@pytest.mark.parametrize("N", [16, 100, 512])
@pytest.mark.parametrize("scale", [1e-6, 1.0, 40.0, 1e6])
def test_root_and_many_radii(S, oracle, N, scale):
    phi = scale * np.stack([oracle.screen(N, max(2.5, N / 40.0), 11 / 3, 3, r) for r in range(3)])
    radii = list(np.linspace(0.0, N / 2.0, 70))
    D, R = S.structure_function(torch.tensor(phi, device="cuda"), 1.0, radii)
    for b in range(3):
        ring, _ = oracle.ring_spectrum(phi[b])
        ref = [oracle.structure_from_spectrum(N, ring, r) for r in radii]
        assert D[b] == pytest.approx(ref, rel=1e-9, abs=1e-9 * max(ref))
        ends = [oracle.structure_from_spectrum(N, ring, r) for r in (1e-3, 0.5 * N)]
        if ends[0] < 1.0 <= ends[1]:
            assert R[b] == pytest.approx(oracle.rdiff_rec(N, ring), rel=1e-9)
        else:
            assert math.isnan(R[b])
