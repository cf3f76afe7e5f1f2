"""The passes that carry transposes (FP32 above 4096: below, fields are stored
by columns and there is none to carry), at 5000 (ragged transpose units of 64
rows by 128 columns, 500-thread row workgroups) and 8000: the pipelined
co-addition, propagation and smear, and the row blocks, equal bit for bit to the
passes without.  Every case asserts from the timing report that the one side
carried transposes and the other did not.

Budgets are chosen so that both sides split the work into the same jobs: one
field of 5000^2 takes 191 MiB, of 8000^2 488; a pipelined job takes four per
screen and wavelength, a plain chunk two and half a one.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

MiB = 1 << 20
LAM = 5e-7


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1301_0514_amd import scint
    scint.load_library()
    return scint


def run(S, call, budget=0):
    """call()'s result and whether a row pass carried transposes."""
    S.set_workspace_budget(budget)
    try:
        S.timing_enable(True)
        out = call()
        torch.cuda.synchronize()
        names = [n for n in S.timing_report() if n.startswith("row_")]
        S.timing_enable(False)
    finally:
        S.set_workspace_budget(0)
    assert names
    return out, any(n.split("_")[1].endswith("T") for n in names)


def geometry(N, n_lambda, seed):
    lam_ref = 650e-9
    z = 2 * np.pi * (N / 12.0) ** 2 / lam_ref
    lams = list(np.linspace(400e-9, 900e-9, n_lambda))
    w = list(np.random.default_rng(seed).uniform(0.5, 2.0, n_lambda))
    return z, lam_ref, lams, w


def poly_pair(S, monkeypatch, N, n_real, n_lambda, bp, bq, seed=1):
    """The co-addition pipelined under budget bp and plain under bq."""
    z, lam_ref, lams, w = geometry(N, n_lambda, seed)
    phi = S.ps_generate(N, 1.0, N / 300.0, 11 / 3, 5 + seed, 0, n_real)

    def call():
        return S.illumination_polychromatic(phi, 1.0, z, lam_ref, lams, w)

    monkeypatch.setenv("SCINT_PIPELINE", "1")
    pl = S.plan_polychromatic(N, n_real, n_lambda, bp or (32 << 30))
    a, carried = run(S, call, bp)
    assert carried and pl["pipelined"]
    monkeypatch.setenv("SCINT_PIPELINE", "0")
    ql = S.plan_polychromatic(N, n_real, n_lambda, bq or (32 << 30))
    b, carried = run(S, call, bq)
    assert not carried and not ql["pipelined"]
    return a, b, pl, ql


# jobs: 12 of two wavelengths; 6 of 2, 2, 1; two realisations a job, the last one
# alone; one wavelength of one realisation a job (4 and 6 jobs)
@pytest.mark.parametrize("N,n_real,n_lambda,bp,bq,jobs", [
    (5000, 3, 8, 1700, 1000, 12), (5000, 2, 5, 1700, 1000, 6), (5000, 5, 2, 3400, 1900, 3),
    (5000, 2, 2, 900, 560, 4), (8000, 2, 3, 2300, 1300, 6)])
def test_pipelined_equals_plain(S, monkeypatch, N, n_real, n_lambda, bp, bq, jobs):
    a, b, pl, ql = poly_pair(S, monkeypatch, N, n_real, n_lambda, bp * MiB, bq * MiB)
    assert pl["n_jobs"] == jobs
    assert (pl["lambdas_per_job"], pl["real_per_job"]) == (ql["lambdas_per_job"], ql["real_per_job"])
    assert torch.equal(a, b)
    assert float(a.mean()) == pytest.approx(1.0, abs=1e-5)


@pytest.mark.parametrize("n_real", [2, 3])
def test_prologue_and_epilogue(S, monkeypatch, n_real):
    # two and three jobs of one realisation
    a, b, pl, _ = poly_pair(S, monkeypatch, 5000, n_real, 2, 1700 * MiB, 1000 * MiB, seed=2)
    assert pl["n_jobs"] == n_real and torch.equal(a, b)


@pytest.mark.parametrize("split,groups", [("0", None), ("1", None), ("0.3", "3:1:5:2"), (None, "1:1:1:1"),
                                          ("0.6", "2:3:1:4")])
def test_split_settings(S, monkeypatch, split, groups):
    # shares of a job's transposes on the x and y passes, and their interleaving
    if split is not None:
        monkeypatch.setenv("SCINT_SIDE_SPLIT", split)
    if groups is not None:
        monkeypatch.setenv("SCINT_SIDE_GROUPS", groups)
    a, b, pl, _ = poly_pair(S, monkeypatch, 5000, 3, 4, 1700 * MiB, 1000 * MiB, seed=3)
    assert pl["n_jobs"] == 6 and torch.equal(a, b)


def test_work_of_one_job_is_split_in_two(S, monkeypatch):
    # by realisations: the sums of the plain loop; by wavelengths: two partial
    # sums, equal to FP32 rounding
    a, b, pl, _ = poly_pair(S, monkeypatch, 5000, 3, 4, 0, 0, seed=4)
    assert pl["n_jobs"] == 2 and torch.equal(a, b)
    a, b, pl, _ = poly_pair(S, monkeypatch, 5000, 1, 5, 0, 0, seed=5)
    assert pl["n_jobs"] == 2 and float((a - b).abs().max()) <= 4e-6 * float(b.abs().max())


@pytest.mark.parametrize("N,n_real,n_lambda", [(5000, 2, 5), (8000, 1, 3)])
def test_x_pass_split_equals_unsplit(S, monkeypatch, N, n_real, n_lambda):
    z, lam_ref, lams, w = geometry(N, n_lambda, N)
    phi = S.ps_generate(N, 1.0, N / 100.0, 11 / 3, 3, 0, n_real)
    out = []
    for parts in ("2", "1"):
        monkeypatch.setenv("SCINT_ITER_SPLIT", parts)
        x, carried = run(S, lambda: S.illumination_polychromatic(phi, 1.0, z, lam_ref, lams, w))
        assert carried
        out.append(x)
    assert torch.equal(*out)


@pytest.mark.parametrize("N,n", [(5000, 3), (8000, 2)])
def test_fresnel_propagate_batches(S, monkeypatch, N, n):
    phi = S.ps_generate(N, 1.0, N / 300.0, 11 / 3, 6, 0, n)
    z = 2 * np.pi * (N / 12.0) ** 2 / LAM
    a, carried = run(S, lambda: S.fresnel_propagate(phi, 1.0, LAM, z, 0.8))
    assert carried
    # a budget below a pipelined pair of jobs: chunks of one screen
    c, _ = run(S, lambda: S.fresnel_propagate(phi, 1.0, LAM, z, 0.8), 3 * N * N * 8)
    monkeypatch.setenv("SCINT_PIPELINE", "0")
    b, carried = run(S, lambda: S.fresnel_propagate(phi, 1.0, LAM, z, 0.8))
    assert not carried
    assert torch.equal(a, b) and torch.equal(c, b)


@pytest.mark.parametrize("n_real,radii", [(4, [3.0]), (5, [2.0, 9.0, 30.0]), (8, [5.0, 20.0])])
def test_smear(S, monkeypatch, n_real, radii):
    N = 5000
    g = torch.Generator(device="cuda").manual_seed(N + n_real)
    I = torch.rand((n_real, N, N), generator=g, device="cuda") + 0.5
    S.source_smear(I[:1].contiguous(), 1.0, radii)  # (the disks' spectra)
    monkeypatch.setenv("SCINT_PIPELINE", "1")
    a, carried = run(S, lambda: S.source_smear(I, 1.0, radii))
    assert carried
    monkeypatch.setenv("SCINT_PIPELINE", "0")
    b, carried = run(S, lambda: S.source_smear(I, 1.0, radii))
    assert not carried and torch.equal(a, b)


# blocks that end inside a screen, and more blocks than a screen has quarters
@pytest.mark.parametrize("N,n", [(5000, 3), (8000, 1)])
def test_row_blocks_of_batches(S, monkeypatch, N, n):
    z = N / LAM  # conjugate planes, for the aperture mode too
    phi = S.ps_generate(N, 1.0, 30.0, 11 / 3, 9, 0, n)
    calls = {
        "generate": lambda: S.ps_generate(N, 1.0, 30.0, 11 / 3, 5, 7, n),
        "screen": lambda: S.ps_screen_fresnel(N, 1.0, 20.0, 11 / 3, 5, LAM, z, n_real=n),
        "screen+phi": lambda: S.ps_screen_fresnel(N, 1.0, 20.0, 11 / 3, 5, LAM, z, n_real=n, want_phi=True,
                                                  want_field=True),
        "field": lambda: S.fresnel_propagate_field(phi, 1.0, LAM, z),
        "aperture": lambda: S.fresnel_aperture(phi, 1.0, LAM, z),
        "structure": lambda: S.structure_function(phi, 1.0, [1.0, 10.0, N / 3.0], want_spectrum=True),
    }
    for name, call in calls.items():
        monkeypatch.setenv("SCINT_SCREEN_JOBS", "1")
        ref, carried = run(S, call)
        assert not carried
        for jobs in ("2", "4", "7"):
            monkeypatch.setenv("SCINT_SCREEN_JOBS", jobs)
            out, carried = run(S, call)
            assert carried, name
            for x, y in zip(out if isinstance(out, tuple) else (out,), ref if isinstance(ref, tuple) else (ref,)):
                assert torch.equal(x, y) if torch.is_tensor(x) else x == y, (name, jobs)


def test_graph_replay_matches_eager(S):
    """Screens, the pipelined co-addition (two jobs) and the pipelined smear in a
    graph: every replay, with eager work and synchronisations between them,
    equals the eager result bit for bit."""
    N, n_real, n_lambda = 5000, 4, 2
    z, lam_ref, lams, w = geometry(N, n_lambda, 6)
    phi = torch.empty((n_real, N, N), dtype=torch.float32, device="cuda")
    I = torch.empty_like(phi)
    ext = torch.empty((n_real, 2, N, N), dtype=torch.float32, device="cuda")

    def step():
        S.ps_generate(N, 1.0, 7.0, 11 / 3, 9, 0, n_real, out=phi)
        S.illumination_polychromatic(phi, 1.0, z, lam_ref, lams, w, out=I)
        S.source_smear(I, 1.0, [5.0, 20.0], out=ext)

    assert S.plan_polychromatic(N, n_real, n_lambda, 5000 * MiB)["n_jobs"] == 2
    try:
        _, carried = run(S, step, 5000 * MiB)  # (the smear's chunk: two pairs)
        assert carried
        S.set_workspace_budget(5000 * MiB)
        g, stream = S.capture_graph(step, warmup=2)
        with torch.cuda.stream(stream):
            step()
        stream.synchronize()
    finally:
        S.set_workspace_budget(0)
    ref = phi.clone(), I.clone(), ext.clone()
    for rep in range(3):
        for t in (phi, I, ext):
            t.fill_(-1.0)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            g.replay()
        stream.synchronize()
        for t, r in zip((phi, I, ext), ref):
            assert torch.equal(t, r), rep
        S.ps_screen_fresnel(128, 1.0, 3.0, 11 / 3, 1, 5e-7, 1e4)
        torch.cuda.synchronize()
