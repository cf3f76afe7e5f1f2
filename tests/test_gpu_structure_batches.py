"""R_diff^rec over batches (ps_structure_function): the levels of bisection per
launch fall with the number of screens, down to one workgroup per screen from
69 on.  Every form takes the same midpoints and decisions, so a screen's root
and D do not depend on its batch; and the time may not grow faster than the
work (with eight levels always, 4096 screens took 46 times as long as 64, with
the rule 7 times).  Roots at either end of the range: the screens are scaled so
that the oracle's D is 1 just inside it, where most levels are needed.
"""
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


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("N,n", [(16, 300), (64, 69), (64, 68), (100, 33), (320, 17), (320, 9)])
def test_root_does_not_depend_on_the_batch(S, N, n, dtype):
    g = torch.Generator(device="cuda").manual_seed(N + n)
    phi = torch.randn((n, N, N), dtype=dtype, device="cuda", generator=g)
    phi *= torch.logspace(-1.0, 1.5, n, device="cuda", dtype=dtype)[:, None, None]  # (the first ones: no root)
    D, R, spec = S.structure_function(phi, 1.0, [1.0, 0.4 * N], want_spectrum=True)
    assert any(math.isnan(r) for r in R) and sum(not math.isnan(r) for r in R) > n // 2
    for b in range(0, n, 4):
        d, r, s = S.structure_function(phi[b:b + 4].contiguous(), 1.0, [1.0, 0.4 * N], want_spectrum=True)
        for j in range(len(r)):
            assert r[j] == R[b + j] or (math.isnan(r[j]) and math.isnan(R[b + j]))
            assert d[j] == D[b + j] and s[j] == spec[b + j]


def test_time_grows_with_the_work(S):
    def best(n):
        phi = torch.randn((n, 64, 64), device="cuda")
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        S.structure_function(phi, 1.0, [1.0])
        t = []
        for _ in range(8):
            a.record()
            S.structure_function(phi, 1.0, [1.0])
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)
    few, many = best(64), best(4096)
    print("64 screens %.3f ms, 4096 %.3f ms" % (few, many))
    assert many < 25 * few


# A screen of one mode, phi = a cos(2 pi k x / N), has power N^2 a^2 / 2 in ring
# k alone, so any root can be set: the highest mode for roots near 1e-3 pixels,
# the lowest for one near N/2 (D grows up to there).
@pytest.mark.parametrize("N,n", [(16, 1), (16, 80), (512, 3), (4096, 1)])
@pytest.mark.parametrize("where", ["1.0001e-3", "2e-3", "0.499 N"])
def test_root_at_the_ends(S, oracle, N, n, where):
    r0 = 0.499 * N if where == "0.499 N" else float(where)
    k = 1 if where == "0.499 N" else N // 2 - 1
    f2 = np.fft.fftfreq(N, 1.0 / N).astype(np.int64) ** 2
    q = 4 * (f2[:, None] + f2[None, :])
    ring = np.zeros(N // 2 + 1)
    ring[k] = N * N / 2.0 / np.count_nonzero((q >= (2 * k - 1) ** 2) & (q < (2 * k + 1) ** 2))
    scale2 = 1.0 / oracle.structure_from_spectrum(N, ring, r0)
    ring *= scale2
    ends = [oracle.structure_from_spectrum(N, ring, r) for r in (1e-3, 0.5 * N)]
    assert ends[0] < 1.0 <= ends[1]  # bracketed
    phi = math.sqrt(scale2) * np.cos(2 * np.pi * (k * np.arange(N) % N) / N)
    t = torch.tensor(phi, device="cuda").expand(n, N, N).contiguous()
    _, R = S.structure_function(t, 1.0)
    ref = oracle.rdiff_rec(N, ring)
    assert ref == pytest.approx(r0, rel=1e-9)
    # near 1e-3 pixels D is the difference of 1 and J0 = 1 - x^2 / 4, x = 2 pi k r / N: a few 2^-53 over
    # x^2 / 4, and half of that for the root; 1e-9 is the bar of the FP64 structure tests
    x = 2 * np.pi * k * r0 / N
    tol = 1e-9 + 4 * 2.0 ** -53 / (x * x / 4)
    for r in R:
        assert r == pytest.approx(ref, rel=tol)
