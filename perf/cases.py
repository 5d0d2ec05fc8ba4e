"""The work that users of the framework have it do, as cases that can be timed and checked.

A case is one call (or the few calls that belong together) on one context: a grid of
``ntheta`` x ``nphi`` rings, ``lmax``, ``P`` separable modes, an arithmetic ``prec`` and,
for most operations, a batch of ``S`` skies.  ``op`` says what is computed:

  beta         filtered maps and beta^hat (``mc`` > 0: minus the Monte-Carlo linear term of
               a finalised state of ``mc`` skies; 0: without a state)
  train        the same through autograd, forward and backward: beta^hat and its gradient
  vjp          the gradient alone
  state        the linear-term state itself: reset, accumulate S skies, finalise
  power        the pair sums of the modal power spectrum
  trispectrum  the quartic sums of the modal trispectrum
  estimator    sample covariance of N vectors, its Cholesky factor, E and sigma^2 of S skies
  theory       the ideal covariance of the modes and alpha of one separable shape

The skies are Gaussian, of the beam-and-noise spectrum that the context filters with; the
mode functions are Legendre polynomials in l and the mask cuts |latitude| < 10 degrees.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1105_2791_amd import ModalContext
from paper_1105_2791_amd.autograd import modal_beta

_SKY_OPS = ("beta", "train", "vjp", "state", "power", "trispectrum")


def _case(op, lmax, ntheta, nphi, P, prec, S, mc=0, N=0):
    return {"op": op, "lmax": lmax, "ntheta": ntheta, "nphi": nphi, "P": P, "prec": prec, "S": S, "mc": mc, "N": N}


def listed():
    def named(name, *a, **k):
        return dict(_case(*a, **k), name=name)
    return [
        # one small sky in double precision, the call of a unit test or a notebook: launches and latency
        named("beta_tiny_f64", "beta", 32, 48, 96, 8, "f64", 1),
        # three skies on a small grid of awkward sizes, odd everywhere, in the fp16 split
        named("beta_ragged_f16x3", "beta", 150, 199, 400, 13, "f16x3", 3, mc=4),
        # the WMAP-size estimator workload in its own arithmetic
        named("beta_wmap500_f32", "beta", 500, 768, 1536, 30, "f32", 8, mc=8),
        # the throughput workload of the benchmark
        named("beta_metric1000_bf16x3", "beta", 1000, 1536, 3072, 40, "bf16x3", 8, mc=8),
        # the largest grid of the mixed batch
        named("beta_mixed2000_bf16x3", "beta", 2000, 3008, 6016, 50, "bf16x3", 4),
        # differentiation through the estimator at the WMAP size, in single precision
        named("train_wmap500_f32", "train", 500, 768, 1536, 30, "f32", 4, mc=8),
        # the gradient at the resolution of the throughput workload
        named("vjp_metric1000_bf16x3", "vjp", 1000, 1536, 3072, 40, "bf16x3", 4, mc=8),
        # building a Monte-Carlo linear-term state
        named("state_500_bf16x3", "state", 500, 768, 1536, 40, "bf16x3", 8),
        # power spectrum of a batch of skies
        named("power_metric1000_bf16x3", "power", 1000, 1536, 3072, 40, "bf16x3", 8),
        # trispectrum with the Monte-Carlo pair means
        named("trispectrum_wmap500_bf16x3", "trispectrum", 500, 768, 1536, 30, "bf16x3", 4, mc=8),
        # covariance from simulations and the estimator with it
        named("estimator_4960", "estimator", 500, 768, 1536, 30, "f32", 8, N=6000),
        # the theory side of a context: ideal covariance and the shape's coefficients
        named("theory_wmap500", "theory", 500, 768, 1536, 30, "f64", 0),
    ]


# a drawn case: the operation, and the ranges of lmax and P it is drawn from
_RANGES = [
    ("beta", 24, 1024, 4, 50), ("beta", 24, 1024, 4, 50), ("beta", 24, 1024, 4, 50), ("train", 24, 512, 4, 36),
    ("vjp", 24, 1000, 4, 44), ("state", 24, 512, 4, 40), ("power", 24, 1024, 4, 44),
    ("trispectrum", 24, 512, 4, 30), ("estimator", 32, 256, 6, 30), ("theory", 24, 512, 4, 30),
]


def _smooth(n):
    """The smallest 5-smooth number >= n: ring lengths are chosen for the transform."""
    while True:
        k = n
        for r in (2, 3, 5):
            while k % r == 0:
                k //= r
        if k == 1:
            return n
        n += 1


def draw(rng):
    op, l0, l1, p0, p1 = _RANGES[rng.randrange(len(_RANGES))]
    lmax = int(round(math.exp(rng.uniform(math.log(l0), math.log(l1)))))
    P = rng.randint(p0, p1)
    ntheta = 3 * lmax // 2 + 1 + rng.randint(0, 8)
    nphi = 2 * _smooth(ntheta)
    if op == "estimator":
        nmax = P * (P + 1) * (P + 2) // 6
        return _case(op, lmax, ntheta, nphi, P, "f32", rng.randint(1, 9), N=int(nmax * rng.uniform(1.2, 2.0)) + 3)
    if op == "theory":
        return _case(op, lmax, ntheta, nphi, P, "f64", 0)
    precs = {"beta": ["bf16x3", "bf16x3", "f16x3", "f32", "f64"], "train": ["f32", "bf16x3"],
             "vjp": ["bf16x3", "f16x3", "f32"], "state": ["bf16x3", "f32"], "power": ["bf16x3", "f32"],
             "trispectrum": ["bf16x3", "f16x3"]}[op]
    prec = precs[rng.randrange(len(precs))]
    if prec == "f64" and lmax > 256:   # double precision serves checks, on smaller grids
        prec = "f32"
    mc = 4 * rng.randint(0, 1) if op in ("beta", "train", "vjp", "trispectrum") else 0
    return _case(op, lmax, ntheta, nphi, P, prec, rng.randint(1, 8 if op != "trispectrum" else 4), mc=mc)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _spectrum(lmax):
    """f_sky (b_l^2 C_l + N_l): a 13' beam, white noise equal to the signal at l = 400."""
    def beam2(l):
        sig = math.radians(13.0 / 60.0) / math.sqrt(8.0 * math.log(2.0))
        return np.exp(-l * (l + 1.0) * sig * sig)
    l = np.arange(lmax + 1, dtype=np.float64)
    cl = np.zeros(lmax + 1)
    noise = float(beam2(np.float64(400.0))) / (400.0 * 401.0)
    cl[2:] = (1.0 - math.sin(math.radians(10.0))) * (beam2(l[2:]) / (l[2:] * (l[2:] + 1.0)) + noise)
    return cl


def _modes(P, lmax):
    return np.ascontiguousarray(np.polynomial.legendre.legvander(2.0 * np.arange(lmax + 1) / lmax - 1.0, P - 1).T)


def _mask(ntheta, nphi):
    lat = np.abs(0.5 * math.pi - (np.arange(ntheta) + 0.75) * math.pi / (ntheta + 0.5))
    return np.repeat((lat >= math.radians(10.0)).astype(np.float64)[:, None], nphi, axis=1)


def _starts(lmax):
    m = np.arange(lmax + 1)
    return m * (2 * lmax + 3 - m) // 2


def _skies(n, lmax, double, gen):
    """a_lm of n Gaussian skies of the spectrum, stored m-major."""
    cl = _spectrum(lmax)
    sd = np.concatenate([np.sqrt(cl[m:] * (1.0 if m == 0 else 0.5)) for m in range(lmax + 1)])
    z = torch.randn((n, sd.size, 2), dtype=torch.float64, device="cuda", generator=gen)
    z *= torch.from_numpy(sd).cuda()[None, :, None]
    z[:, :lmax + 1, 1] = 0.0
    return torch.view_as_complex(z).to(torch.complex128 if double else torch.complex64)


def _sky_inputs(case, seed):
    """The skies analysed, the Monte-Carlo skies of the state, and the cotangents."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    double = case["prec"] == "f64"
    alm = _skies(case["S"], case["lmax"], double, gen)
    sims = _skies(case["mc"], case["lmax"], double, gen) if case["mc"] else None
    cot = None
    if case["op"] in ("train", "vjp"):
        cot = torch.randn((case["S"], _nmax(case["P"])), dtype=torch.float64, device="cuda", generator=gen)
    return alm, sims, cot


def _vector_inputs(case, seed):
    """beta^hat vectors with a few strong directions, alpha and the skies to estimate on."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n, N, S = _nmax(case["P"]), case["N"], case["S"]
    kw = {"dtype": torch.float64, "device": "cuda", "generator": gen}
    u = torch.randn((4, n), **kw) / math.sqrt(n)
    u *= torch.tensor([14.0, 11.0, 9.0, 7.0], dtype=torch.float64, device="cuda")[:, None]
    def rows(k):
        return math.sqrt(6.0) * (torch.randn((k, n), **kw) + torch.randn((k, 4), **kw) @ u)
    b = rows(N)
    return b, torch.randn((n,), **kw), rows(S)


def _terms(lmax, seed):
    """A local-type shape, C_l C_l' + permutations, of a seeded amplitude and tilt."""
    r = np.random.RandomState(seed % (1 << 31))
    l = np.arange(lmax + 1, dtype=np.float64)
    x = np.zeros(lmax + 1)
    x[2:] = (l[2:] * (l[2:] + 1.0)) ** -(1.0 + 0.02 * r.randn())
    return (1.0 + 0.1 * r.rand()) * np.stack([x, x, np.ones(lmax + 1)])[None]


def _weights(case, seed):
    """The whitened spectrum c_l of the sky that the ideal covariance is taken for."""
    c = 1.0 + 0.05 * np.random.RandomState((seed + 1) % (1 << 31)).rand(case["lmax"] + 1)
    c[:2] = 0.0
    return c


def prepare(case, seed):
    lmax, P = case["lmax"], case["P"]
    mask = _mask(case["ntheta"], case["nphi"]) if case["op"] in _SKY_OPS else None
    ctx = ModalContext(lmax, case["ntheta"], case["nphi"], P, case["prec"], _modes(P, lmax), _spectrum(lmax), mask)
    st = {"op": case["op"], "ctx": ctx}
    if case["op"] == "theory":
        st["c"], st["terms"] = _weights(case, seed), _terms(lmax, seed)
    elif case["op"] == "estimator":
        st["b"], st["alpha"], st["data"] = _vector_inputs(case, seed)
    else:
        st["alm"], sims, st["cot"] = _sky_inputs(case, seed)
        st["state"] = None
        if case["op"] == "train":
            st["alm"].requires_grad_(True)
        if case["op"] == "state" or case["mc"]:
            st["state"] = ctx.linear_state()
        if case["mc"]:
            ctx.linear_reset(st["state"])
            ctx.linear_accumulate(st["state"], sims)
            ctx.linear_finalize(st["state"])
    return st


def run(st):
    op, ctx = st["op"], st["ctx"]
    if op == "beta":
        return ctx.beta(st["alm"], state=st["state"])
    if op == "train":
        beta = modal_beta(st["alm"], ctx, st["state"])
        (grad,) = torch.autograd.grad(beta, st["alm"], st["cot"])
        return {"beta": beta.detach(), "grad": grad}
    if op == "vjp":
        return ctx.beta_vjp(st["alm"], st["cot"], state=st["state"])
    if op == "state":
        s = st["state"]
        ctx.linear_reset(s)
        ctx.linear_accumulate(s, st["alm"])
        ctx.linear_finalize(s)
        v = ctx.pair_means(s)
        at = -(-v.numel() * v.element_size() // 256) * 256   # Z follows V, 256-byte aligned
        nz = ctx.npairs * ctx.nalm * 2 * v.element_size()
        return {"V": v, "Z": s[at:at + nz].view(ctx.complex_dtype).view(ctx.npairs, ctx.nalm)}
    if op == "power":
        return ctx.power_beta(st["alm"], state=st["state"])
    if op == "trispectrum":
        return ctx.trispectrum(st["alm"], state=st["state"])
    if op == "estimator":
        zeta = ctx.covariance_sample(st["b"])
        E, s2 = ctx.fnl(zeta, st["alpha"], st["data"])
        return {"zeta": zeta, "E": E, "sigma2": s2}
    return {"zeta0": ctx.ideal_covariance(st["c"]), "alpha": ctx.alpha_separable(st["terms"])}


# ---------------------------------------------------------------------------
# the work that cannot be done without
# ---------------------------------------------------------------------------

def _nmax(P):
    return P * (P + 1) * (P + 2) // 6


def work(case):
    lmax, P, S, op = case["lmax"], case["P"], case["S"], case["op"]
    nalm, npairs, nmax = (lmax + 1) * (lmax + 2) // 2, P * (P + 1) // 2, _nmax(P)
    npix, real = case["ntheta"] * case["nphi"], 8 if case["prec"] == "f64" else 4
    if op == "estimator":
        return {"bytes": 8.0 * (case["N"] * nmax + nmax * nmax + (S + 1) * nmax),
                "flops": case["N"] * nmax * (nmax + 1.0) + nmax ** 3 / 3.0 + 2.0 * (S + 1) * nmax ** 2}
    if op == "theory":
        nmu = (3 * lmax + 2) // 2
        # sums over the nodes of the products of three Q_ab(mu), a <= b: each distinct one once
        return {"bytes": 8.0 * (nmax * nmax + nmax + P * (lmax + 1)),
                "flops": 2.0 * nmu * min(_nmax(npairs), 3.5 * nmax * (nmax + 1)) + 2.0 * nmu * npairs * (lmax + 1)}
    maps = S * P * (2.0 * nalm * case["ntheta"] + 2.5 * npix * math.log2(case["nphi"]))
    alm, Z, V = S * nalm * 2 * real, npairs * nalm * 2 * real, npairs * npix * real
    lin = 4.0 * S * npairs * nalm + 2.0 * S * npairs * P * (lmax + 1) if case["mc"] else 0.0
    cubic = 2.0 * S * nmax * npix
    if op == "beta":
        return {"bytes": alm + 8.0 * S * nmax + (Z if case["mc"] else 0), "flops": maps + cubic + lin}
    if op in ("train", "vjp"):
        fwd = cubic + lin if op == "train" else 0.0
        return {"bytes": 2.0 * alm + 8.0 * S * nmax + (Z if case["mc"] else 0),
                "flops": 2 * maps + fwd + 2.0 * S * npix * P * npairs + lin}
    if op == "state":
        return {"bytes": alm + V + Z, "flops": maps + 2.0 * S * npairs * npix
                + npairs * (2.0 * nalm * case["ntheta"] + 2.5 * npix * math.log2(case["nphi"]))}
    if op == "power":
        return {"bytes": alm + 8.0 * S * npairs, "flops": maps + 2.0 * S * npairs * npix}
    nquad = P * (P + 1) * (P + 2) * (P + 3) // 24
    # with pair means the mixed term V_ab M_c M_d needs every product of two pairs
    cells = npairs * (npairs + 1) / 2.0 if case["mc"] else nquad
    return {"bytes": alm + 8.0 * S * nquad + (V if case["mc"] else 0), "flops": maps + 2.0 * S * cells * npix}


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------

def _gauss_legendre(n):
    """Nodes (descending) and weights, in extended precision until the end."""
    z = np.cos(np.longdouble(math.pi) * (np.arange(n, dtype=np.longdouble) + 0.75) / (n + 0.5))
    for it in range(7):
        p1, p2 = np.ones_like(z), np.zeros_like(z)
        for j in range(1, n + 1):
            p1, p2 = ((2 * j - 1) * z * p1 - (j - 1) * p2) / np.longdouble(j), p1
        dp = n * (z * p1 - p2) / (z * z - 1)
        if it < 6:
            z = z - p1 / dp
    return z.astype(np.float64), (2 / ((1 - z * z) * dp * dp)).astype(np.float64)


def _lambda_rows(x, lmax, m0, m1):
    """lambda_lm(x) for m0 <= m < m1, as [l][m - m0][x]; scaled by powers of 2^300 on the way up."""
    big = 2.0 ** 300
    m = torch.arange(m0, m1, dtype=torch.float64, device="cuda")
    k = np.arange(1, max(m1, 2))
    cum = np.concatenate([[0.0], np.cumsum(np.log((2.0 * k - 1.0) / (2.0 * k)))])[m0:m1]
    pref = torch.from_numpy(0.5 * (np.log((2.0 * np.arange(m0, m1) + 1.0) / (4.0 * math.pi)) + cum)).cuda()
    log_seed = pref[:, None] + m[:, None] * (0.5 * torch.log1p(-x * x))[None]
    n = torch.clamp(torch.floor(-log_seed / math.log(big)), min=0.0)       # lambda = value 2^(-300 n)
    sign = torch.where(m.long() % 2 == 0, 1.0, -1.0)[:, None]
    seed = sign * torch.exp(log_seed + n * math.log(big))
    cur, prev, one = torch.zeros_like(seed), torch.zeros_like(seed), torch.ones((), dtype=torch.float64, device="cuda")
    out = torch.zeros((lmax + 1, m1 - m0, x.numel()), dtype=torch.float64, device="cuda")
    for l in range(m0, lmax + 1):
        a = torch.zeros(m1 - m0, dtype=torch.float64, device="cuda")
        b = torch.zeros_like(a)
        hi = min(l, m1) - m0            # rows with m < l step, the row m = l starts
        mm = m[:hi]
        a[:hi] = torch.sqrt((4.0 * l * l - 1.0) / (l * l - mm * mm))
        b[:hi] = a[:hi] * torch.sqrt(((l - 1.0) ** 2 - mm * mm) / (4.0 * (l - 1.0) ** 2 - 1.0))
        new = a[:, None] * (x * cur) - b[:, None] * prev
        if l < m1:
            new[l - m0] = seed[l - m0]
        prev, cur = cur, new
        over = (cur.abs() > 2.0 ** 100) & (n > 0)   # what n > 0 still hides is below 2^-200
        f = torch.where(over, one / big, one)
        cur, prev, n = cur * f, prev * f, n - over.double()
        out[l] = torch.where(n == 0, cur, 0.0)
    return out


class _Sphere:
    """The grid of a case in 64 bits: weights, lambda, transforms."""

    def __init__(self, case):
        self.lmax, self.nt, self.nphi, self.P = case["lmax"], case["ntheta"], case["nphi"], case["P"]
        x, w = _gauss_legendre(self.nt)
        self.x = torch.from_numpy(x).cuda()
        self.w = torch.from_numpy(w * 2.0 * math.pi / self.nphi).cuda()[:, None] * \
            torch.from_numpy(_mask(self.nt, self.nphi)).cuda()
        cl, q = _spectrum(self.lmax), _modes(self.P, self.lmax)
        self.qw = torch.from_numpy(np.where(cl > 0, q / np.sqrt(np.where(cl > 0, cl, 1.0)), 0.0)).cuda()
        self.at = _starts(self.lmax)
        self.nrp = (self.nt + 1) // 2
        ab = torch.triu_indices(self.P, self.P, device="cuda")
        self.a, self.b = ab[0], ab[1]
        self.rings = max(1, (1 << 28) // (self.nphi * max(1, self.a.numel())))

    def _lambda(self):
        step = max(1, min(64, int(3e9 / (8.0 * (self.lmax + 1) * self.nrp))))
        for m0 in range(0, self.lmax + 1, step):
            m1 = min(self.lmax + 1, m0 + step)
            lam = _lambda_rows(self.x[:self.nrp], self.lmax, m0, m1)
            for m in range(m0, m1):
                yield m, lam[m:, m - m0].contiguous()

    def spectra(self, alm):
        """Ring coefficients [S P][ring][m] of the filtered maps."""
        S, P = alm.shape[0], self.P
        F = torch.empty((S * P, self.nt, self.lmax + 1), dtype=torch.complex128, device="cuda")
        for m, lam in self._lambda():
            n = self.lmax + 1 - m
            a = alm[:, self.at[m]:self.at[m] + n].to(torch.complex128)
            c = torch.view_as_real(self.qw[None, :, m:] * a[:, None])           # [S][P][l][2]
            c = c.permute(0, 1, 3, 2).reshape(S * P * 2, n)
            e, o = c[:, ::2] @ lam[::2], c[:, 1::2] @ lam[1::2]
            north, south = (e + o).view(S * P, 2, -1), (e - o).view(S * P, 2, -1)
            F[:, :self.nrp, m] = torch.complex(north[:, 0].contiguous(), north[:, 1].contiguous())
            ns = self.nt - self.nrp
            s = torch.flip(south[:, :, :ns], (2,))
            F[:, self.nrp:, m] = torch.complex(s[:, 0].contiguous(), s[:, 1].contiguous())
        return F

    def bands(self, *spectra):
        """Runs of rings: (first, last, pixel weights, the maps [S][P][pixels] of each spectrum)."""
        for r0 in range(0, self.nt, self.rings):
            r1 = min(self.nt, r0 + self.rings)
            maps = [None if F is None else
                    (torch.fft.irfft(F[:, r0:r1].contiguous(), n=self.nphi) * self.nphi).reshape(
                        -1, self.P, (r1 - r0) * self.nphi) for F in spectra]
            yield (r0, r1, self.w[r0:r1].reshape(-1), *maps)

    def pair_mean(self, M):
        """The mean over the skies of M of the products of each pair [pairs][pixels]."""
        V = torch.zeros((self.a.numel(), M.shape[2]), dtype=torch.float64, device="cuda")
        for s in range(M.shape[0]):
            V += M[s][self.a] * M[s][self.b]
        return V / M.shape[0]

    def adjoint(self, rows):
        """sum over the grid of rows lambda_lm e^(-i m phi), [row][nalm]; rows(r0, r1) gives a band."""
        first = rows(0, 1)
        G = torch.empty((first.shape[0], self.nt, self.lmax + 1), dtype=torch.complex128, device="cuda")
        for r0 in range(0, self.nt, self.rings):
            r1 = min(self.nt, r0 + self.rings)
            G[:, r0:r1] = torch.fft.rfft(rows(r0, r1).view(-1, r1 - r0, self.nphi))[:, :, :self.lmax + 1]
        return self.adjoint_spectra(G)

    def adjoint_spectra(self, G):
        out = torch.empty((G.shape[0], (self.lmax + 1) * (self.lmax + 2) // 2), dtype=torch.complex128, device="cuda")
        ns = self.nt - self.nrp
        for m, lam in self._lambda():
            g = G[:, :, m]
            north, south = g[:, :self.nrp], torch.zeros_like(g[:, :self.nrp])
            south[:, :ns] = torch.flip(g[:, self.nrp:], (1,))
            n = self.lmax + 1 - m
            res = torch.empty((G.shape[0], n, 2), dtype=torch.float64, device="cuda")
            for par, h in ((0, north + south), (1, north - south)):
                if lam[par::2].shape[0]:
                    for k, part in ((0, h.real), (1, h.imag)):
                        res[:, par::2, k] = part.contiguous() @ lam[par::2].t().contiguous()
            out[:, self.at[m]:self.at[m] + n] = torch.view_as_complex(res)
        return out

    def fold(self, g):
        """c_m = 2 - delta_m0, and no imaginary part for m = 0."""
        g = 2.0 * g
        g[:, :self.lmax + 1] = torch.complex(0.5 * g[:, :self.lmax + 1].real, torch.zeros_like(g[:, :self.lmax + 1].real))
        return g


def _triples(P):
    t = [(p, r, s) for p in range(P) for r in range(p, P) for s in range(r, P)]
    return torch.tensor(t, device="cuda").t()


def _pair_index(P):
    ix = np.zeros((P, P), dtype=np.int64)
    a, b = np.triu_indices(P)
    ix[a, b] = ix[b, a] = np.arange(a.size)
    return torch.from_numpy(ix).cuda()


def _exact_beta(sp, F, Fmc):
    S, P = F.shape[0] // sp.P, sp.P
    E = torch.zeros((S, sp.a.numel(), P), dtype=torch.float64, device="cuda")
    L = torch.zeros_like(E)
    for _, _, w, M, Mmc in sp.bands(F, Fmc):
        V = None if Mmc is None else w * sp.pair_mean(Mmc)
        for s in range(S):
            Mt = M[s].t().contiguous()
            E[s] += (w * M[s][sp.a] * M[s][sp.b]) @ Mt
            if V is not None:
                L[s] += V @ Mt
    p, r, s = _triples(P)
    ix = _pair_index(P)
    return E[:, ix[p, r], s] - (L[:, ix[p, r], s] + L[:, ix[p, s], r] + L[:, ix[r, s], p])


def _exact_vjp(sp, F, Fmc, cot):
    """G_t = 3 w sum_ab C_tab (M_a M_b - V_ab), C the symmetric tensor of the cotangent."""
    S, P = F.shape[0] // sp.P, sp.P
    p, r, s = _triples(P)
    C = torch.zeros((S, P, P, P), dtype=torch.float64, device="cuda")
    perms = {(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)}
    t = (p, r, s)
    same = (p == r).long() + (r == s).long()
    count = torch.tensor([6.0, 3.0, 1.0], dtype=torch.float64, device="cuda")[same]
    for a, b, c in perms:
        C[:, t[a], t[b], t[c]] = cot / count
    K = C[:, :, sp.a, sp.b] * torch.where(sp.a == sp.b, 3.0, 6.0)
    G = torch.empty((S * P, sp.nt, sp.lmax + 1), dtype=torch.complex128, device="cuda")
    for r0, r1, w, M, Mmc in sp.bands(F, Fmc):
        V = 0.0 if Mmc is None else sp.pair_mean(Mmc)
        for s in range(S):
            g = w * (K[s] @ (M[s][sp.a] * M[s][sp.b] - V))
            G[s * P:(s + 1) * P, r0:r1] = torch.fft.rfft(g.view(P, r1 - r0, sp.nphi))[:, :, :sp.lmax + 1]
    z = sp.adjoint_spectra(G).view(S, P, -1)
    q = torch.cat([sp.qw[:, m:] for m in range(sp.lmax + 1)], 1)
    return sp.fold((z * q).sum(1))


def _exact_state(sp, F):
    V = torch.empty((sp.a.numel(), sp.nt, sp.nphi), dtype=torch.float64, device="cuda")
    for r0, r1, w, M in sp.bands(F):
        V[:, r0:r1] = sp.pair_mean(M).view(-1, r1 - r0, sp.nphi)
    Z = sp.fold(sp.adjoint(lambda r0, r1: (V[:, r0:r1] * sp.w[r0:r1]).contiguous()))
    return {"V": V, "Z": Z}


def _exact_quartic(sp, F, Fmc):
    S, P, n = F.shape[0] // sp.P, sp.P, sp.a.numel()
    K = torch.zeros((S, n, n), dtype=torch.float64, device="cuda")
    for _, _, w, M, Mmc in sp.bands(F, Fmc):
        V = None if Mmc is None else sp.pair_mean(Mmc)
        for s in range(S):
            B = M[s][sp.a] * M[s][sp.b]
            if V is None:
                K[s] += (w * B) @ B.t()
            else:   # M M M M - 3 (V MM + MM V) + 3 V V; the mean over the pairings leaves 6 and 3
                A = B - 3.0 * V
                K[s] += (w * A) @ A.t() - 6.0 * ((w * V) @ V.t())
    ix = _pair_index(P).cpu().numpy()
    p, r, s, u = np.array([(p, r, s, u) for p in range(P) for r in range(p, P) for s in range(r, P)
                           for u in range(s, P)]).T
    pick = [(torch.from_numpy(ix[i, j]).cuda(), torch.from_numpy(ix[k, l]).cuda())
            for i, j, k, l in ((p, r, s, u), (p, s, r, u), (p, u, r, s))]
    return sum(K[:, i, j] for i, j in pick) / 3.0


def _exact_theory(case, seed):
    lmax, P = case["lmax"], case["P"]
    x, w = _gauss_legendre((3 * lmax + 2) // 2)
    x, w = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    leg = torch.empty((lmax + 1, x.numel()), dtype=torch.float64, device="cuda")
    leg[0], leg[1] = 1.0, x
    for l in range(2, lmax + 1):
        leg[l] = ((2 * l - 1) * x * leg[l - 1] - (l - 1) * leg[l - 2]) / l
    leg *= (2.0 * torch.arange(lmax + 1, device="cuda") + 1.0)[:, None]
    q = torch.from_numpy(_modes(P, lmax)).cuda()
    cl = torch.from_numpy(_spectrum(lmax)).cuda()
    a, b = torch.triu_indices(P, P, device="cuda")
    c = torch.from_numpy(_weights(case, seed)).cuda()
    Q = (c * q[a] * q[b]) @ leg                                       # [pairs][nodes]
    ix, (p, r, s), n = _pair_index(P), _triples(P), _nmax(P)
    zeta = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    T = torch.stack([((w * Q[i]) * Q) @ Q.t() for i in range(Q.shape[0])])
    for row in range(0, n, 512):
        i, j, k = (t[row:row + 512, None] for t in (p, r, s))
        for d, e, f in ((p, r, s), (p, s, r), (r, p, s), (r, s, p), (s, p, r), (s, r, p)):
            zeta[row:row + 512] += T[ix[i, d[None]], ix[j, e[None]], ix[k, f[None]]]
    zeta /= 48.0 * math.pi
    qw = torch.where(cl > 0, q / torch.sqrt(torch.where(cl > 0, cl, 1.0)), 0.0)
    alpha = torch.zeros(n, dtype=torch.float64, device="cuda")
    for X, Y, Z in torch.from_numpy(_terms(lmax, seed)).cuda():
        x3 = [(u * qw) @ leg for u in (X, Y, Z)]
        for i, j, k in ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)):
            alpha += (x3[i][p] * x3[j][r] * x3[k][s]) @ w
    return {"zeta0": zeta, "alpha": alpha / (48.0 * math.pi)}


def _exact_estimator(case, seed):
    b, alpha, data = _vector_inputs(case, seed)
    zeta = b.t() @ b / (6.0 * case["N"])
    L = torch.linalg.cholesky(zeta.cpu())
    y = torch.linalg.solve_triangular(L, torch.cat([alpha[None], data]).cpu().t().contiguous(), upper=False)
    yy = (y[:, 0] @ y[:, 0]).item()
    return {"zeta": zeta, "E": ((y[:, 0] @ y[:, 1:]) / yy).numpy(), "sigma2": 6.0 / yy}


def exact(case, seed):
    op = case["op"]
    if op == "estimator":
        return _exact_estimator(case, seed)
    if op == "theory":
        return _exact_theory(case, seed)
    alm, sims, cot = _sky_inputs(case, seed)
    sp = _Sphere(case)
    F = sp.spectra(alm)
    Fmc = None if sims is None else sp.spectra(sims)
    if op == "beta":
        return _exact_beta(sp, F, Fmc)
    if op == "train":
        return {"beta": _exact_beta(sp, F, Fmc), "grad": _exact_vjp(sp, F, Fmc, cot)}
    if op == "vjp":
        return _exact_vjp(sp, F, Fmc, cot)
    if op == "state":
        return _exact_state(sp, F)
    if op == "power":
        out = torch.zeros((alm.shape[0], sp.a.numel()), dtype=torch.float64, device="cuda")
        for _, _, w, M in sp.bands(F):
            for s in range(M.shape[0]):
                K = (w * M[s]) @ M[s].t().contiguous()
                out[s] += K[sp.a, sp.b]
        return out
    return _exact_quartic(sp, F, Fmc)
