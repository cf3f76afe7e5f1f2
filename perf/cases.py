"""What a user of this framework has it do, as cases that can be timed.

Each case is one pass of a program through the public entry points of
paper_1301_0514_amd.scint: screens, propagation, co-addition over a passband,
extended sources, gradients and the observables, from a 256^2 double-precision
pattern up to the batched 8192^2 step and the 20000^2 K_s band.  listed() are
fixed ones, draw() gives more of the same ranges, prepare() makes what the
program has in hand before the call, run() is the pass, work() the bytes and
operations the pass cannot do without, and exact() the outputs in 64 bits from
the formulas (Habibi, Moniez, Ansari & Rahvar, A&A 2013), in plain torch.
Lengths are in pixels (pixel side 1); the wavelength is a label and
z = 2 pi rho^2 / lambda sets the Fresnel radius rho.
"""
import math

import torch

from paper_1301_0514_amd import scint

LAM = 650e-9  # metres; enters only through lambda z
BETA = 11.0 / 3.0
PI = math.pi


def listed():
    return [
        # the plain method in double precision, R_F = 32 px, R_diff = 4 px: the
        # smallest call, where launches and latency count
        dict(name="plain_f64_256", kind="screen", N=256, n=1, f64=True, rho=32.0, R=4.0, beta=BETA, want_phi=True),
        # a few small given screens seen at one wavelength (an interactive look at a configuration)
        dict(name="propagate_f32_640x3", kind="propagate", N=640, n=3, f64=False, rho=20.0, R=6.0, beta=BETA,
             scale=1.0),
        # one step of a fit of small screens through torch.autograd: pattern and its gradient
        dict(name="autograd_f32_1000x4", kind="autograd", N=1000, n=4, f64=False, rho=30.0, R=12.0, beta=BETA,
             scale=0.9),
        # one pattern of a 4096^2 screen, strong regime: the ordinary single-wavelength call
        dict(name="single_f32_4096", kind="screen", N=4096, n=1, f64=False, rho=64.0, R=8.0, beta=BETA,
             want_phi=False),
        # one pattern at the paper's scale, a length with factors of five
        dict(name="paper_f32_10000", kind="screen", N=10000, n=1, f64=False, rho=100.0, R=30.0, beta=3.2,
             want_phi=False),
        # the differentiation workload: screens, patterns, loss against targets, adjoint from the kept field
        dict(name="grad_f32_2048x16", kind="grad", N=2048, n=16, f64=False, rho=48.0, R=24.0, beta=BETA),
        # a weighted passband (a filter curve) over two ordinary screens
        dict(name="poly_f32_2000x2x9", kind="poly", N=2000, n=2, f64=False, rho=60.0, R=16.0, beta=BETA, n_lam=9,
             band=0.25, weighted=True),
        # the paper's 20000^2 screen through the K_s band in 21 wavelengths: the longest row
        dict(name="ks_f32_20000x21", kind="poly", N=20000, n=1, f64=False, rho=57.5, R=4.42, beta=BETA, n_lam=21,
             band=0.0463, weighted=False),
        # the batched step: 8 screens, 32 wavelengths over 400-900 nm, four stellar disks: the largest
        dict(name="step_f32_8192x8x32", kind="step", N=8192, n=8, f64=False, rho=90.0, R=30.0, beta=BETA, n_lam=32,
             band=0.385, n_r=4, r_max=360.0),
        # stellar disks over a few given patterns, an odd number of them
        dict(name="smear_f32_1280x5x3", kind="smear", N=1280, n=5, f64=False, n_r=3, r_max=80.0),
        # the paper's own one-FFT numerics with its window, at the conjugate planes
        dict(name="aperture_f32_4096x2", kind="aperture", N=4096, n=2, f64=False, widen=1.0, R=20.0, beta=BETA,
             margin=10.0),
        # the observables of two simulated screens and their patterns: modulation index (whole and fiducial
        # zone), light curves, structure function
        dict(name="observe_f32_4000x2", kind="observe", N=4000, n=2, f64=False, R=14.0, beta=BETA, n_lines=48,
             n_samples=5000, mode=1, n_r=8),
    ]


# kind: its share of the draws, the largest N in single and in double precision, and the most
# points x wavelengths of one case
RANGES = {
    "screen": (4, 16384, 4096, 3e8),
    "propagate": (3, 16384, 4096, 3e8),
    "autograd": (2, 4096, 1280, 7e7),
    "grad": (2, 4096, 1280, 7e7),
    "poly": (3, 20000, 2048, 8e9),
    "step": (2, 8192, 1024, 4e9),
    "smear": (2, 8192, 2048, 2e8),
    "aperture": (2, 16384, 2560, 3e8),
    "observe": (2, 8192, 4000, 1.4e8),
}


def draw(rng):
    """One more case: a kind by its share, N from the supported sizes spread over their logarithm, the rest within
    the ranges that the listed cases stand for."""
    kinds = list(RANGES)
    kind = rng.choices(kinds, [RANGES[k][0] for k in kinds])[0]
    f64 = rng.random() < 0.2
    most = RANGES[kind][3] / (8 if f64 else 1)
    hi = RANGES[kind][2 if f64 else 1]
    lo = 128 if kind in ("aperture", "observe") else 64
    sizes = [N for N in scint.supported_sizes(torch.float64 if f64 else torch.float32) if lo <= N <= hi]
    target = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    N = min(sizes, key=lambda s: abs(math.log(s / target)))
    n_lam = rng.randint(2, 40) if kind in ("poly", "step") else 1
    n_lam = max(2, min(n_lam, int(most / N ** 2))) if n_lam > 1 else 1
    n_r = rng.randint(1, 5)
    per = N * N * n_lam * (n_r if kind == "smear" else 1)
    n = max(1, min(int(math.exp(rng.uniform(0.0, math.log(17.0)))), int(most / per)))
    R = math.exp(rng.uniform(math.log(3.0), math.log(max(6.0, N / 200.0))))
    rho = math.exp(rng.uniform(math.log(4.0), math.log(max(8.0, min(128.0, N / 10.0)))))
    beta = rng.choice([3.1, 3.2, BETA, 3.9])
    c = dict(kind=kind, N=N, n=n, f64=f64)
    if kind == "screen":
        c.update(rho=rho, R=R, beta=beta, want_phi=rng.random() < 0.5)
    elif kind in ("propagate", "autograd"):
        c.update(rho=rho, R=R, beta=beta, scale=rng.uniform(0.7, 1.4))
    elif kind == "grad":
        c.update(rho=rho, R=max(R, N / 200.0), beta=beta)
    elif kind == "poly":
        c.update(rho=rho, R=R, beta=beta, n_lam=n_lam, band=rng.uniform(0.03, 0.4), weighted=rng.random() < 0.5)
    elif kind == "step":
        c.update(rho=rho, R=R, beta=beta, n_lam=n_lam, band=rng.uniform(0.03, 0.4), n_r=n_r,
                 r_max=rng.uniform(2.0, N / 8.0))
    elif kind == "smear":
        c.update(n_r=n_r, r_max=rng.uniform(2.0, N / 8.0))
    elif kind == "aperture":
        c.update(widen=rng.uniform(1.0, 1.6), R=max(R, 8.0), beta=beta,
                 margin=rng.uniform(0.0, min(10.0, 0.24 * math.sqrt(2 * PI * N))))
    else:
        c.update(R=R, beta=beta, n_lines=rng.randint(1, 64), n_samples=rng.randint(N // 4, 2 * N),
                 mode=rng.randint(0, 1), n_r=rng.randint(1, 12))
    return c


# ---------------------------------------------------------------- inputs
def _dtype(case):
    return torch.float64 if case["f64"] else torch.float32


def _spectrum_const(R, beta):
    """S(q) = const * q^-beta (cycles per pixel), with R in pixels (Sect. 3.1, Eq. spectre)."""
    f = 2.0 ** -beta * beta * math.gamma(-beta / 2) / math.gamma(beta / 2)
    return R ** (2.0 - beta) / (2.0 * (2.0 * PI) ** (beta - 1.0) * f)


def _freq(N):
    return torch.fft.fftfreq(N, 1.0 / N, dtype=torch.float64, device="cuda")


def _sqrt_spectrum(N, R, beta):
    k = _freq(N)
    k2 = k[:, None] ** 2 + k[None, :] ** 2
    k2[0, 0] = 1.0
    a = (_spectrum_const(R, beta) * float(N) ** beta) ** 0.5 / N * k2.pow_(-beta / 4)
    a[0, 0] = 0.0
    return a


def _screens(N, n, R, beta, gen):
    """n phase screens [n, N, N] in float64 from torch's generator."""
    out = torch.empty((n, N, N), dtype=torch.float64, device="cuda")
    amp = _sqrt_spectrum(N, R, beta)
    for b in range(n):
        c = torch.randn((N, N), dtype=torch.complex128, device="cuda", generator=gen)  # unit variance in all
        out[b] = torch.fft.ifft2(c.mul_(amp), norm="forward").real
        del c
    return out.mul_(math.sqrt(2.0))


def _patterns(N, n, gen):
    """n speckled patterns of mean 1."""
    phi = _screens(N, n, 0.02 * N, BETA, gen)
    return torch.stack([_field(p, 0.05 * N).abs().square() for p in phi])


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _z(rho, lam=LAM):
    return 2.0 * PI * rho ** 2 / lam


def _lambdas(case):
    h, n = case["band"], case["n_lam"]
    return [LAM * (1.0 - h + 2.0 * h * j / (n - 1)) for j in range(n)]


def _weights(case):
    """A filter curve, lower towards the ends of the band."""
    n = case["n_lam"]
    return [0.2 + math.sin(PI * (j + 0.5) / n) for j in range(n)] if case.get("weighted") else None


def _radii(case):
    n = case["n_r"]
    return [case["r_max"] * 2.0 ** -j for j in range(n)][::-1]


def _aperture_z(case):
    return case["widen"] * case["N"] / LAM


def _lines(case, seed):
    r = torch.Generator().manual_seed(int(seed) + 1)
    u = torch.rand((case["n_lines"], 4), generator=r, dtype=torch.float64)
    return [[float(a * case["N"]), float(b * case["N"]), float(0.3 + c), float(2 * d - 1)] for a, b, c, d in u]


def _structure_radii(case):
    n = case["n_r"]
    return [case["R"] * 2.0 ** (j / 2.0 - 2.0) for j in range(n)]


def prepare(case, seed):
    N, n, dt, kind = case["N"], case["n"], _dtype(case), case["kind"]
    st = dict(case, seed=int(seed))
    gen = _gen(seed)
    if kind in ("propagate", "poly", "autograd", "aperture", "observe"):
        st["phi"] = _screens(N, n, case["R"], case["beta"], gen).to(dt)
    if kind == "autograd":
        st["phi"].requires_grad_()
        st["grad_I"] = torch.randn((n, N, N), dtype=dt, device="cuda", generator=gen)
    if kind == "grad":
        st["target"] = _patterns(N, n, gen).to(dt)
    if kind in ("smear", "observe"):
        st["I"] = _patterns(N, n, gen).to(dt)
    if kind == "observe":
        st["lines"] = _lines(case, seed)
    if kind == "step":  # the step's arrays, kept by the program
        st["phi"] = torch.empty((n, N, N), dtype=dt, device="cuda")
        st["I"] = torch.empty_like(st["phi"])
        st["I_ext"] = torch.empty((n, case["n_r"], N, N), dtype=dt, device="cuda")
    return st


def run(st):
    N, n, dt, kind = st["N"], st["n"], _dtype(st), st["kind"]
    if kind == "screen":
        return scint.ps_screen_fresnel(N, 1.0, st["R"], st["beta"], st["seed"], LAM, _z(st["rho"]), n_real=n,
                                       dtype=dt, want_phi=st["want_phi"])
    if kind == "propagate":
        return scint.fresnel_propagate(st["phi"], 1.0, LAM, _z(st["rho"]), st["scale"])
    if kind == "autograd":
        I = scint.fresnel_intensity(st["phi"], 1.0, LAM, _z(st["rho"]), st["scale"])
        return I.detach(), torch.autograd.grad(I, st["phi"], st["grad_I"])[0]
    if kind == "grad":
        z = _z(st["rho"])
        I, phi, field = scint.ps_screen_fresnel(N, 1.0, st["R"], st["beta"], st["seed"], LAM, z, n_real=n, dtype=dt,
                                                want_phi=True, want_field=True)
        loss, grad_I = scint.ps_l2_loss(I, st["target"])
        grad = scint.fresnel_propagate_vjp(phi, 1.0, LAM, z, grad_I, field=field)
        return I, grad, torch.tensor(loss)
    if kind == "poly":
        return scint.illumination_polychromatic(st["phi"], 1.0, _z(st["rho"]), LAM, _lambdas(st), _weights(st))
    if kind == "step":
        scint.ps_generate(N, 1.0, st["R"], st["beta"], st["seed"], 0, n, out=st["phi"])
        scint.illumination_polychromatic(st["phi"], 1.0, _z(st["rho"]), LAM, _lambdas(st), out=st["I"])
        scint.source_smear(st["I"], 1.0, _radii(st), out=st["I_ext"])
        return st["phi"], st["I"], st["I_ext"]
    if kind == "smear":
        return scint.source_smear(st["I"], 1.0, _radii(st))
    if kind == "aperture":
        return scint.fresnel_aperture(st["phi"], 1.0, LAM, _aperture_z(st), margin_rf=st["margin"])
    m, mean = scint.ps_modulation_index(st["I"], want_mean=True)
    q = N // 8
    m_zone = scint.ps_modulation_index_region(st["I"], q, q, N - 2 * q, N - 2 * q)
    curves, m_curves = scint.light_curves(st["I"], st["lines"], st["n_samples"], st["mode"])
    D, R_rec, S = scint.structure_function(st["phi"], 1.0, _structure_radii(st), want_spectrum=True)
    return {"m": torch.tensor(m), "mean": torch.tensor(mean), "m_zone": torch.tensor(m_zone), "curves": curves,
            "m_curves": torch.tensor(m_curves), "D": torch.tensor(D), "R": torch.tensor(R_rec), "S": torch.tensor(S)}


# ---------------------------------------------------------------- work
def work(case):
    """Each input read once and each output written once; operations of the transforms (5 M log2 M per complex
    transform of M points) and of the products with the transfer function."""
    N, n, kind = case["N"], case["n"], case["kind"]
    rb = 8 if case["f64"] else 4
    pts = float(N) * N * n
    fft = 10.0 * math.log2(N) * pts  # one 2-D transform of the batch
    prop = 2 * fft + 20.0 * pts      # exp(i s phi), transform, transfer function, inverse transform, |.|^2
    if kind == "screen":
        return {"bytes": pts * rb * (2 if case["want_phi"] else 1), "flops": fft + prop}
    if kind == "propagate":
        return {"bytes": 2 * pts * rb, "flops": prop}
    if kind == "autograd":  # phi, grad_I; pattern, gradient
        return {"bytes": 4 * pts * rb, "flops": 2 * prop}
    if kind == "grad":  # target; pattern, gradient
        return {"bytes": 3 * pts * rb, "flops": fft + 2 * prop}
    if kind == "poly":
        return {"bytes": 2 * pts * rb, "flops": case["n_lam"] * prop}
    smear = (0.5 + 0.5 * case["n_r"]) * fft if "n_r" in case else 0.0  # real patterns: half a complex transform
    if kind == "step":
        return {"bytes": (2 + case["n_r"]) * pts * rb, "flops": fft + case["n_lam"] * prop + smear}
    if kind == "smear":
        return {"bytes": (1 + case["n_r"]) * pts * rb, "flops": smear}
    if kind == "aperture":
        return {"bytes": 2 * pts * rb, "flops": fft + 20.0 * pts}
    curve = float(n) * case["n_lines"] * case["n_samples"]
    return {"bytes": 2 * pts * rb + curve * rb * (1 + (4 if case["mode"] else 1)), "flops": 0.5 * fft + 12.0 * pts}


# ---------------------------------------------------------------- the same in 64 bits
_MASK = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11) on int64 tensors that hold 32-bit words."""
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((p1 >> 32) & _MASK) ^ c1 ^ k0, p1 & _MASK, ((p0 >> 32) & _MASK) ^ c3 ^ k1, p0 & _MASK)
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return c0, c1, c2, c3


def _exact_screen(N, R, beta, seed, r):
    """Screen r of a seed: complex normals from Philox at counter (kx, ky, r, 0), the spectrum, inverse transform."""
    k = torch.arange(N, dtype=torch.int64, device="cuda")
    kx, ky = k[None, :].expand(N, N), k[:, None].expand(N, N)
    zero = torch.zeros((), dtype=torch.int64, device="cuda")
    w0, w1, w2, w3 = _philox(kx, ky, zero + r, zero, seed & _MASK, (seed >> 32) & _MASK)
    u1 = ((w0 << 21 | w1 >> 11).double() + 0.5) * 2.0 ** -53
    u2 = ((w2 << 21 | w3 >> 11).double() + 0.5) * 2.0 ** -53
    del w0, w1, w2, w3
    rad = u1.log_().mul_(-2.0).sqrt_().mul_(_sqrt_spectrum(N, R, beta))
    c = torch.polar(rad, u2.mul_(2.0 * PI))
    return torch.fft.ifft2(c, norm="forward").real  # sqrt(2) Re sum c g / sqrt(2)


def _transfer(N, rho, conj=False):
    k = _freq(N)
    turns = PI * rho ** 2 * k ** 2 / float(N) ** 2
    return torch.polar(torch.ones_like(k), (1.0 if conj else -1.0) * 2.0 * PI * (turns - turns.round()))


def _through(u, h):
    """ifft2(H fft2(u)) with H = h(ky) h(kx); u is given up."""
    f = torch.fft.fft2(u)
    del u
    f.mul_(h[:, None]).mul_(h[None, :])
    return torch.fft.ifft2(f)


def _unit(phi, scale=1.0):
    return torch.polar(torch.ones((), dtype=torch.float64, device="cuda").expand_as(phi), phi.double() * scale)


def _field(phi, rho, scale=1.0):
    return _through(_unit(phi, scale), _transfer(phi.shape[-1], rho))


def _intensity(phi, rho, scale=1.0):
    return _field(phi, rho, scale).abs().square()


def _gradient(phi, rho, scale, grad_I):
    """dL/dphi for dL/dI = grad_I."""
    N = phi.shape[-1]
    g = _through(2.0 * grad_I.double() * _field(phi, rho, scale), _transfer(N, rho, conj=True))
    return scale * (g * _unit(phi, scale).conj()).imag


def _coadded(phi, rho, lams, weights):
    w = weights or [1.0] * len(lams)
    out = torch.zeros(phi.shape, dtype=torch.float64, device="cuda")
    for lam, wj in zip(lams, w):
        out.add_(_intensity(phi, rho * math.sqrt(lam / LAM), LAM / lam), alpha=wj / sum(w))
    return out


def _smeared(I, radii):
    N = I.shape[-1]
    k = _freq(N)
    d2 = k[:, None] ** 2 + k[None, :] ** 2
    F = torch.fft.fft2(I.double())
    out = []
    for r in radii:
        P = (d2 <= r * r).double()
        out.append(torch.fft.ifft2(F * torch.fft.fft2(P / P.sum())).real)
    return torch.stack(out)


def _aperture(phi, z, margin):
    N = phi.shape[-1]
    rho2 = LAM * z / (2.0 * PI)
    j = torch.arange(N, dtype=torch.float64, device="cuda")
    Lm, x = margin * math.sqrt(rho2), j + 0.5
    w = torch.ones_like(j)
    if Lm > 0.0:
        w = torch.where(x <= Lm, 0.5 * (1.0 - torch.cos(PI * x / Lm)), w)
        w = torch.where(x >= N - Lm, 0.5 * (1.0 + torch.cos(PI * (x - N + Lm) / Lm)), w)
    a = torch.polar(w, (j - N // 2) ** 2 / (2.0 * rho2))
    G = _unit(phi).mul_(a[:, None]).mul_(a[None, :])
    return torch.fft.fftshift(torch.fft.fft2(G)).abs().square() / (2.0 * PI * rho2) ** 2


def _curves(I, lines, n_samples, mode):
    N = I.shape[-1]
    p = torch.tensor(lines, dtype=torch.float64, device="cuda")
    k = torch.arange(n_samples, dtype=torch.float64, device="cuda")
    x, y = p[:, 0:1] + k * p[:, 2:3], p[:, 1:2] + k * p[:, 3:4]
    at = lambda yy, xx: I[..., yy.long() % N, xx.long() % N].double()  # noqa: E731
    if mode == 0:
        return at(torch.floor(y + 0.5), torch.floor(x + 0.5))
    ix, iy = torch.floor(x), torch.floor(y)
    fx, fy = x - ix, y - iy
    return ((1 - fx) * (1 - fy) * at(iy, ix) + fx * (1 - fy) * at(iy, ix + 1) + (1 - fx) * fy * at(iy + 1, ix)
            + fx * fy * at(iy + 1, ix + 1))


def _index(I, dims):
    mean = I.double().mean(dims)
    return I.double().std(dims, correction=0) / mean, mean


def _structure(phi, radii):
    """Ring spectrum, D_rec at the radii and the r with D_rec(r) = 1 (Sect. 3.1.1)."""
    N = phi.shape[-1]
    k = _freq(N)
    ring = torch.floor(((4.0 * (k[:, None] ** 2 + k[None, :] ** 2)).sqrt() + 1.0) / 2.0).long().flatten()
    power = torch.fft.fft2(phi.double()).abs().square().flatten() / float(N) ** 2
    S = (torch.bincount(ring, power) / torch.bincount(ring))[:N // 2 + 1]
    q = torch.arange(N // 2 + 1, dtype=torch.float64, device="cuda") / N

    def D(r):
        return float((q * S * (1.0 - torch.special.bessel_j0(2.0 * PI * q * r))).sum() * 4.0 * PI / N)

    lo, hi = 1e-3, 0.5 * N
    if not (D(lo) < 1.0 <= D(hi)):
        return [D(r) for r in radii], math.nan, S
    while hi - lo > 1e-12 * hi:
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if D(mid) < 1.0 else (lo, mid)
    return [D(r) for r in radii], 0.5 * (lo + hi), S


def exact(case, seed):
    st = prepare(case, seed)
    N, n, kind = case["N"], case["n"], case["kind"]
    if kind in ("screen", "grad", "step"):
        phi = torch.stack([_exact_screen(N, case["R"], case["beta"], int(seed), r) for r in range(n)])
    if kind == "screen":
        I = torch.stack([_intensity(p, case["rho"]) for p in phi])
        return (I, phi) if case["want_phi"] else I
    if kind == "propagate":
        return torch.stack([_intensity(p, case["rho"], case["scale"]) for p in st["phi"]])
    if kind == "autograd":
        ps = st["phi"].detach()
        return (torch.stack([_intensity(p, case["rho"], case["scale"]) for p in ps]),
                torch.stack([_gradient(p, case["rho"], case["scale"], g) for p, g in zip(ps, st["grad_I"])]))
    if kind == "grad":
        I = torch.stack([_intensity(p, case["rho"]) for p in phi])
        d = I - st["target"].double()
        grad = torch.stack([_gradient(p, case["rho"], 1.0, 2.0 * x) for p, x in zip(phi, d)])
        return I, grad, d.square().sum((1, 2))
    if kind == "poly":
        return torch.stack([_coadded(p, case["rho"], _lambdas(case), _weights(case)) for p in st["phi"]])
    if kind == "step":
        I = torch.stack([_coadded(p, case["rho"], _lambdas(case), None) for p in phi])
        return phi, I, torch.stack([_smeared(i, _radii(case)) for i in I])
    if kind == "smear":
        return torch.stack([_smeared(i, _radii(case)) for i in st["I"]])
    if kind == "aperture":
        return torch.stack([_aperture(p, _aperture_z(case), case["margin"]) for p in st["phi"]])
    q = N // 8
    m, mean = _index(st["I"], (1, 2))
    m_zone = _index(st["I"][:, q:N - q, q:N - q], (1, 2))[0]
    curves = _curves(st["I"], st["lines"], case["n_samples"], case["mode"])
    found = [_structure(p, _structure_radii(case)) for p in st["phi"]]
    return {"m": m, "mean": mean, "m_zone": m_zone, "curves": curves, "m_curves": _index(curves, (2,))[0],
            "D": torch.tensor([f[0] for f in found], dtype=torch.float64),
            "R": torch.tensor([f[1] for f in found], dtype=torch.float64), "S": torch.stack([f[2] for f in found])}
