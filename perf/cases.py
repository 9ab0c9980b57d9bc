"""Performance cases of the sGW/sROI library: what its users run, by size.

Every case calls the public entry points of ``paper_2601_21005_amd.sgw`` on
the synthetic systems of ``paper_2601_21005_amd.systems``: H-capped Si
clusters with Kleinman-Bylander projectors, and Gaussian wells without.  A
case's ``op`` names the path: ``hpsi`` (one Hamiltonian application),
``lanczos`` (spectral interval of a new system), ``filter`` (Chebyshev
occupied-space filter of white noise), ``propagate`` (e^{-iHt} of stochastic
orbitals), ``tdh`` (linear-response substeps), ``sigma`` (the whole
Sigma_c(t) estimate), ``features`` (control-variate features of white noise)
and ``train`` (the control-variate network, forward, backward and Adam).

``exact`` restates each operation in plain 64-bit torch.
"""
import math

import numpy as np
import torch

from paper_2601_21005_amd import sgw, systems

PREC = {"c64": sgw.SGW_C64, "c128": sgw.SGW_C128, "c64_bf16x2": sgw.SGW_C64_BF16X2KB}
ECUT = 28.0
# encloses the spectrum of every cluster below (their rigorous lower bounds
# lie above -16 Ha, T is clipped at 28 Ha and V_loc and V_NL are attractive)
INTERVAL = (-16.0, 28.5)
WELL_BETA = 50.0


def listed():
    return [
        # one orbital of a small cluster: residuals, single-state checks; all
        # launches and latency (40^3: 8 x 8 x 8 projector tiles)
        dict(name="hpsi 40 1 vector", op="hpsi", n=40, n_si=17, prec="c64", nvec=1),
        # the H application of the subspace iteration and of the headline
        # Gpt*vec/s figure on the benchmark's 64^3 Si35H36-shaped cluster
        dict(name="hpsi 64 256 vectors", op="hpsi", n=64, n_si=35, prec="c64", nvec=256),
        # FP64 reference runs on the larger clusters of the uneven batch
        dict(name="hpsi 96 c128", op="hpsi", n=96, n_si=147, prec="c128", nvec=20),
        # the 128^3 cluster shape of the precision study, 1632 projectors
        dict(name="hpsi 128", op="hpsi", n=128, n_si=357, prec="c64", nvec=48),
        # spectral interval, the first thing run on a new system
        dict(name="lanczos 64", op="lanczos", n=64, n_si=35, prec="c64", steps=60),
        # Chebyshev filter at the benchmark's batch: 8 samples x 65 real
        # vectors, two per complex vector (a stretch of its 1338 terms)
        dict(name="filter 64 260 vectors", op="filter", n=64, n_si=35, prec="c64", nvec=260,
             terms=40),
        # zeta orbitals of 8 samples over two output steps
        dict(name="propagate 64 16 vectors", op="propagate", n=64, n_si=35, prec="c64", nvec=16,
             dt=0.05, steps=2),
        # linear response at the benchmark's batch: 8 samples x 64 orbitals
        # with their tangent copies, 1024 vectors
        dict(name="tdh 64 8x64", op="tdh", n=64, n_si=35, prec="c64", ns=8, neta=64, nsub=4,
             dt=0.05),
        # the reduced-precision form on a larger box with few orbitals
        dict(name="tdh 96 bf16x2 4x16", op="tdh", n=96, n_si=71, prec="c64_bf16x2", ns=4,
             neta=16, nsub=2, dt=0.05),
        # the whole estimate: the 32^3 Gaussian wells in FP64 (time axis and
        # filter shortened)
        dict(name="sigma 32 wells c128", op="sigma", n=32, n_si=0, prec="c128", ns=8, neta=8,
             n_tau=20, dt=0.2, m_sub=4, terms=300, n_xi=10000),
        # one chunk of cheap samples for the control variate's mean
        dict(name="features 64 16384", op="features", n=64, states=64, samples=16384),
        # the control variate's network on its training set
        dict(name="train 1536", op="train", samples=1536, steps=10),
    ]


# clusters by grid length (h = 0.6 bohr except the 64^3 benchmark cluster)
_CLUSTERS = {16: (0,), 24: (0, 5), 32: (0, 5), 40: (5, 17), 48: (17, 29), 56: (29, 35),
             64: (35, 47), 80: (47, 71), 96: (71, 147), 112: (99, 147), 128: (147,)}


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["hpsi", "hpsi", "hpsi", "lanczos", "filter", "filter", "propagate", "tdh",
                     "tdh", "sigma", "features", "train"])
    if op == "train":
        return dict(op=op, samples=_log_int(rng, 150, 4096), steps=rng.randint(5, 12))
    if op == "features":
        n = rng.choice([16, 24, 32, 40, 48, 64])
        most = min(65536, 16384 * 64 ** 3 // n ** 3)
        return dict(op=op, n=n, states=rng.choice([8, 17, 32, 48, 64]),
                    samples=_log_int(rng, 100, most))
    if op == "sigma":
        n = rng.choice([16, 24, 32])
        return dict(op=op, n=n, n_si=0, prec="c128", ns=rng.randint(1, 8),
                    neta=rng.choice([2, 4, 8]), n_tau=rng.randint(5, 20), dt=0.2,
                    m_sub=rng.choice([1, 2, 4]), terms=rng.randint(100, 300),
                    n_xi=_log_int(rng, 1000, 10000))
    n = rng.choice(sorted(k for k in _CLUSTERS if k >= (24 if op == "tdh" else 16)))
    if op == "tdh":
        n = min(n, 96)
    n_si = rng.choice([s for s in _CLUSTERS[n] if op != "tdh" or s <= 71])
    prec = rng.choice(["c64", "c64", "c128"] if n_si == 0 else
                      ["c64", "c64", "c64_bf16x2", "c128"])
    case = dict(op=op, n=n, n_si=n_si, prec=prec)
    # points x vectors no larger than the benchmark's, FP64 a quarter of it
    most = (64 ** 3) // (4 if prec == "c128" else 1)
    if op == "hpsi":
        case["nvec"] = _log_int(rng, 1, max(1, min(1024, 256 * most // n ** 3)))
    elif op == "lanczos":
        case["steps"] = rng.randint(20, 60)
    elif op == "filter":
        case.update(nvec=_log_int(rng, 4, max(4, min(512, 200 * most // n ** 3))),
                    terms=rng.randint(20, 40))
    elif op == "propagate":
        case.update(nvec=2 * _log_int(rng, 1, max(1, min(32, 24 * most // n ** 3))),
                    dt=rng.choice([0.05, 0.1, 0.2]), steps=rng.randint(1, 2))
    else:
        orbitals = max(4, min(512, 400 * most // n ** 3))
        neta = rng.choice([k for k in (2, 4, 8, 16, 32, 64) if k <= max(2, orbitals)])
        case.update(neta=neta, ns=_log_int(rng, 1, max(1, min(32, orbitals // neta))),
                    nsub=rng.randint(1, 3), dt=0.05)
    return case


# ------------------------------------------------------------------ inputs
def _system(case):
    n, n_si = case["n"], case["n_si"]
    if n_si == 0:
        return systems.gaussian_wells(seed=1010, n=n, h=0.5)
    species, pos = systems.si_cluster(n_si, seed=1002)
    h = 0.5 if (n, n_si) == (64, 35) else 0.6
    return systems.cluster_model(species, pos, n=n, h=h, ecut=ECUT)


_kept = {}


def _context(case, nvec):
    """The context of the case's system: a program creates it once and uses
    it for every batch (only the last one is kept here)."""
    key = (case["n"], case["n_si"], case["prec"], nvec)
    if key not in _kept:
        _kept.clear()
        s = _system(case)
        _kept[key] = s, sgw.Context(s.grid.n, s.grid.h, s.v_loc, s.projectors,
                                    precision=PREC[case["prec"]], ecut=s.ecut, max_nvec=nvec)
    return _kept[key]


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _noise(g, nvec, N, dV):
    """Complex vectors of two real +-1/sqrt(dV) white-noise orbitals each."""
    b = torch.randint(0, 2, (nvec, N, 2), generator=g, device="cuda", dtype=torch.int8)
    return torch.view_as_complex((2.0 * b.float() - 1.0) / math.sqrt(dV))


def _smooth(g, count, n, h, width=0.8):
    """Real orbitals: white noise smoothed over ``width`` bohr, unit norm
    (float32, device)."""
    k = 2 * math.pi * torch.fft.fftfreq(n, d=h, device="cuda")
    w = torch.exp(-0.5 * width ** 2 * k * k)
    out = torch.empty((count, n ** 3), device="cuda")
    for i in range(0, count, 64):
        m = min(64, count - i)
        x = torch.randn((m, n, n, n), generator=g, device="cuda")
        x = torch.fft.fftn(x, dim=(1, 2, 3)) * (w[:, None, None] * w[None, :, None] * w)
        x = torch.fft.ifftn(x, dim=(1, 2, 3)).real.reshape(m, -1)
        out[i:i + m] = x / (x.norm(dim=1, keepdim=True) * h ** 1.5)
    return out


def _orbital(case, seed):
    """A normalised real orbital in the middle of the box (host, FP64)."""
    s = _system(case)
    rs = np.random.default_rng(seed)
    d = systems.grid_coords(s.grid) - 0.5 * s.grid.L + rs.uniform(-0.5, 0.5, 3)
    phi = np.exp(-np.sum(d * d, axis=1) / (2 * 2.0 ** 2)) * (1 + 0.5 * np.sin(d @ rs.normal(size=3)))
    return phi / np.sqrt(np.sum(phi * phi) * s.grid.h ** 3)


def _tdh_inputs(case, seed):
    """Occupied-like real orbitals with the norms of a filtered noise set, and
    the kick potential."""
    n, h = case["n"], _system(case).grid.h
    g = _gen(seed)
    eta = _smooth(g, case["ns"] * case["neta"], n, h) * 8.0
    dv = _smooth(g, case["ns"], n, h, width=1.5) * 20.0
    return eta.reshape(case["ns"], case["neta"], -1), dv


def _features_inputs(case, seed):
    return _smooth(_gen(seed), case["states"], case["n"], 0.5)


def _train_inputs(case, seed):
    g = _gen(seed)
    n = case["samples"]
    x = torch.randn((n, 64), generator=g, device="cuda").square()   # |<phi|zeta>|^2
    y = torch.tanh(x[:, :8] - 1).sum(1) * 0.4 + 0.5 * torch.randn(n, generator=g, device="cuda")
    return x, y, x.double().mean(0).cpu().numpy(), x.double().std(0).cpu().numpy()


def prepare(case, seed):
    op = case["op"]
    if op == "train":
        x, y, mean, std = _train_inputs(case, seed)
        net = sgw.Mlp(systems.mlp_init(seed % 1000))
        net.set_standardization(mean, std)
        return dict(case=case, net=net, x=x, y=y)
    if op == "features":
        wells = dict(case, n_si=0, prec="c64")
        _, ctx = _context(wells, 1)
        return dict(case=case, ctx=ctx, phi=_features_inputs(case, seed), seed=seed,
                    out=torch.empty((case["samples"], case["states"]), device="cuda"))
    nvec = {"lanczos": 1, "sigma": 64}.get(op) or (
        2 * case["ns"] * case["neta"] if op == "tdh" else case["nvec"])
    s, ctx = _context(case, nvec)
    st = dict(case=case, ctx=ctx, seed=seed)
    if op in ("hpsi", "propagate"):
        st["x"] = torch.randn((nvec, ctx.N), generator=_gen(seed), device="cuda",
                              dtype=torch.complex64).to(ctx.cdtype)
        if op == "hpsi":
            st["y"] = torch.empty_like(st["x"])
    elif op == "filter":
        st["x"] = _noise(_gen(seed), nvec, ctx.N, s.grid.h ** 3).to(ctx.cdtype)
        st["v"] = torch.empty_like(st["x"])
        st["coef"] = sgw.sgw_gapped_coefficients(*_gap(case), 1e-7, *_interval(case),
                                                 case["terms"])
    elif op == "tdh":
        ns, neta = case["ns"], case["neta"]
        eta, dv = _tdh_inputs(case, seed)
        psi = ctx.vectors(nvec).view(ns, 2, neta, ctx.N)
        psi[:, 0] = eta
        st["psi"], st["v"], st["u"] = psi, ctx.fields(ns), ctx.fields(ns)
        st["st"] = ctx.tdh_state(psi, st["v"], st["u"], ctx.fields(ns), ns, neta, 2.0 / neta)
        ctx.tdh_init(st["st"], dv.to(ctx.rdtype).contiguous())
    elif op == "sigma":
        st["phi"] = _orbital(case, seed)
    return st


def run(st):
    case, op = st["case"], st["case"]["op"]
    if op == "hpsi":
        st["ctx"].apply_H(st["x"], st["y"])
        return st["y"]
    if op == "lanczos":
        return st["ctx"].lanczos_bounds(case["steps"], seed=st["seed"], pad=0.01)
    if op == "filter":
        st["v"].copy_(st["x"])
        st["ctx"].fermi_filter(st["v"], st["coef"], *_interval(case))
        return st["v"]
    if op == "propagate":
        st["ctx"].cheb_propagate(st["x"], case["dt"], case["steps"], *_interval(case))
        return st["x"]
    if op == "tdh":
        st["ctx"].tdh_step(st["st"], case["nsub"], case["dt"])
        return [st["psi"], st["v"], st["u"]]
    if op == "sigma":
        sig, x, _ = st["ctx"].sigma_estimate(st["phi"], **_sigma_params(case, st["seed"]))
        return [sig, x]
    if op == "features":
        return sgw.cv_features(st["ctx"], st["phi"], st["seed"], 0, case["samples"], st["out"])
    # the network works in 32 bits; its parameters and losses come back in
    # 64-bit host arrays
    hist = st["net"].train(st["x"], st["y"], case["steps"], lr=1e-3)
    return [st["net"].params().astype(np.float32), hist.astype(np.float32)]


def _interval(case):
    """Clusters: INTERVAL; wells (no kinetic cutoff): [-V, T_max]."""
    if case["n_si"]:
        return INTERVAL
    s = _system(case)
    tmax = 1.5 * (math.pi / s.grid.h) ** 2
    return float(s.v_loc.min()) - 1.0, tmax + 1.0


def _gap(case):
    """The filter's band edges."""
    return (-4.86, -4.44) if case["n_si"] else (-0.46, -0.13)


def _sigma_params(case, seed):
    emin, emax = _interval(case)
    return dict(seed=seed, n_zeta=case["ns"], n_eta=case["neta"], n_tau=case["n_tau"],
                dt=case["dt"], m_sub=case["m_sub"], ncoef=case["terms"], emin=emin, emax=emax,
                mu=-0.3, beta=WELL_BETA, n_xi=case["n_xi"], f_g=0.003)


# ------------------------------------------------------------------ work
def _nnz(case):
    """Projector values of the system (spheres of 6 r_c)."""
    if not case["n_si"]:
        return 0
    s = _system(case)
    rc = s.projectors.rc
    return float(np.sum(np.minimum(s.grid.N, 4 / 3 * math.pi * (6 * rc / s.grid.h) ** 3)))


def work(case):
    op = case["op"]
    if op == "train":
        n, p = case["samples"], 64 * 256 + 256 * 256
        return {"bytes": 4.0 * (n * 65 + 2 * p), "flops": 6.0 * n * p * case["steps"]}
    N = case["n"] ** 3
    if op == "features":
        return {"bytes": 4.0 * (case["states"] * N + case["samples"] * case["states"]),
                "flops": 2.0 * case["states"] * N * case["samples"]}
    c = 16 if case["prec"] == "c128" else 8
    nnz, fft = _nnz(case), 5.0 * N * math.log2(N)
    h_flops = 2 * fft + 8.0 * N + 8.0 * nnz
    if op == "sigma":
        ns, neta, nt = case["ns"], case["neta"], case["n_tau"]
        filt = case["terms"] * ns * (1 + neta) / 2 * h_flops
        tdh = nt * case["m_sub"] * ns * (2 * neta * (2 * fft + 16.0 * N) + 2 * fft)
        zeta = nt * 30 * 2 * ns * h_flops / 2
        return {"bytes": 8.0 * N + 16.0 * ns * (2 * nt + 1), "flops": filt + tdh + zeta}
    if op == "lanczos":
        return {"bytes": 8.0 * N + c * N, "flops": case["steps"] * (h_flops + 20.0 * N)}
    if op == "tdh":
        nv = 2 * case["ns"] * case["neta"]
        return {"bytes": 2.0 * c * N * nv + 4.0 * c * N * case["ns"],
                "flops": case["nsub"] * nv * (2 * fft + 24.0 * N + 16.0 * nnz)}
    if op == "hpsi":
        terms = 1
    elif op == "filter":
        terms = case["terms"] - 1
    else:
        lo, hi = _interval(case)
        terms = case["steps"] * (0.5 * (hi - lo) * case["dt"] + 14)
    return {"bytes": 2.0 * c * N * case["nvec"] + 0.5 * c * (N + nnz),
            "flops": terms * case["nvec"] * h_flops}


# ------------------------------------------------------------------ exact, 64 bits
_M64 = (1 << 64) - 1


def _s64(v):
    v &= _M64
    return v - (1 << 64) if v >> 63 else v


def _shr(z, k):
    return (z >> k) & ((1 << (64 - k)) - 1)


def _sm64(x):
    """SplitMix64's output for counters x (int64 tensor, wrapping)."""
    z = x + _s64(0x9E3779B97F4A7C15)
    z = (z ^ _shr(z, 30)) * _s64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _s64(0x94D049BB133111EB)
    return z ^ _shr(z, 31)


def _words(seed, kind, sample, l, count):
    """Words 0 .. count - 1 of random stream (kind, sample, l)."""
    t = torch.tensor([(kind << 40) | (sample << 20) | l], dtype=torch.int64, device="cuda")
    key = _sm64(_sm64(t) ^ seed)
    return _sm64(key + torch.arange(count, device="cuda"))


def _signs(seed, kind, sample, l, N):
    w = _words(seed, kind, sample, l, (N + 63) // 64)
    bits = (w[:, None] >> torch.arange(64, device="cuda")) & 1
    return (1 - 2 * bits).reshape(-1)[:N].double()


class _Exact:
    """H, the split-step pieces and the Chebyshev maps in complex FP64."""

    def __init__(self, case):
        s = _system(case)
        n, h = s.grid.n, s.grid.h
        self.n, self.N, self.h, self.dV = n, s.grid.N, h, h ** 3
        self.v = torch.from_numpy(s.v_loc).cuda()
        k = 2 * math.pi * torch.fft.fftfreq(n, d=h, device="cuda", dtype=torch.float64)
        k2 = (k * k)[:, None, None] + (k * k)[None, :, None] + k * k
        T = 0.5 * k2
        self.T = T.clamp(max=s.ecut) if s.ecut > 0 else T
        self.coul = torch.where(k2 > 0, 4 * math.pi / k2.clamp(min=1e-300), torch.zeros_like(k2))
        self.B = None
        if s.projectors is not None:
            self._projectors(s.projectors)

    def _projectors(self, p):
        n, h, L = self.n, self.h, self.n * self.h
        i = h * torch.arange(n, device="cuda", dtype=torch.float64)
        self.E = torch.from_numpy(p.ekb).cuda()
        self.B = torch.empty((p.nproj, self.N), dtype=torch.float64, device="cuda")
        for q, a in enumerate(p.atom_of):
            d = [torch.remainder(i - float(p.pos[a][x]) + 0.5 * L, L) - 0.5 * L for x in range(3)]
            dx, dy, dz = d[0][None, None, :], d[1][None, :, None], d[2][:, None, None]
            d2 = dx * dx + dy * dy + dz * dz
            rc = float(p.rc[q])
            f = torch.exp(-d2 / (2 * rc * rc))
            if p.l[q] == 1:
                f = f * (dx, dy, dz)[int(p.m[q])]
            f = torch.where(d2 <= (p.rcut_over_rc * rc) ** 2, f, torch.zeros_like(f)).reshape(-1)
            self.B[q] = f / torch.sqrt((f * f).sum() * self.dV)

    def mult(self, x, m):
        """F^-1 m F x for x [..., N]."""
        sh = x.shape
        y = torch.fft.fftn(x.reshape(-1, self.n, self.n, self.n), dim=(1, 2, 3)) * m
        return torch.fft.ifftn(y, dim=(1, 2, 3)).reshape(sh)

    def project(self, x):
        """<beta_p|x_v> as [P][nv]."""
        r = torch.view_as_real(x.reshape(-1, self.N)).permute(1, 0, 2).reshape(self.N, -1)
        c = self.B @ r
        return self.dV * torch.view_as_complex(c.reshape(c.shape[0], -1, 2).contiguous())

    def spread(self, c):
        """sum_p beta_p c_pv as [nv][N]."""
        r = torch.view_as_real(c.contiguous()).reshape(c.shape[0], -1)
        y = (self.B.t() @ r).reshape(self.N, -1, 2).permute(1, 0, 2).contiguous()
        return torch.view_as_complex(y)

    def apply(self, x):
        y = self.mult(x, self.T) + self.v * x
        if self.B is not None:
            y += self.spread(self.E[:, None] * self.project(x)).reshape(x.shape)
        return y

    def series(self, coef, lo, hi, x):
        c, R = 0.5 * (hi + lo), 0.5 * (hi - lo)
        a, out = x, coef[0] * x
        if len(coef) > 1:
            b = (self.apply(x) - c * x) / R
            out = out + coef[1] * b
            for k in coef[2:]:
                a, b = b, 2 * (self.apply(b) - c * b) / R - a
                out += k * b
        return out

    def kb_exponential(self, tau):
        """K with exp(-i tau V_NL) = 1 + B K <B|."""
        P = self.B.shape[0]
        S = self.dV * (self.B @ self.B.t())
        m = torch.zeros((2 * P, 2 * P), dtype=torch.complex128, device="cuda")
        m[:P, :P] = -1j * tau * S * self.E
        m[:P, P:] = torch.eye(P, dtype=torch.complex128, device="cuda")
        return -1j * tau * self.E[:, None] * torch.linalg.matrix_exp(m)[:P, P:]

    def tdh(self, eta, dv, weight):
        """State (psi [S][2][L][N], v, u, vh0) after the kick."""
        psi = torch.stack([eta.to(torch.complex128), -1j * dv[:, None] * eta], dim=1)
        self.vh0 = self.mult(self.density(psi, weight)[0] + 0j, self.coul).real
        v = self.v.expand(eta.shape[0], -1).clone()
        return psi, v, torch.zeros_like(v)

    def density(self, psi, w):
        e, d = psi[:, 0], psi[:, 1]
        return w * (e.abs() ** 2).sum(1), 2 * w * (e.conj() * d).real.sum(1)

    def local(self, psi, v, u, a):
        ph = torch.exp(-1j * a * v)[:, None]
        d = ph * (psi[:, 1] - 1j * a * u[:, None] * psi[:, 0])
        return torch.stack([ph * psi[:, 0], d], dim=1)

    def substep(self, psi, v, u, tau, w, K):
        psi = self.local(psi, v, u, 0.5 * tau)
        kb = (lambda p: p + self.spread(K @ self.project(p)).reshape(p.shape)) if K is not None \
            else (lambda p: p)
        psi = kb(self.mult(kb(psi), torch.exp(-1j * tau * self.T)))
        rho, drho = self.density(psi, w)
        v = self.v + self.mult(rho + 0j, self.coul).real - self.vh0
        u = self.mult(drho + 0j, self.coul).real
        return self.local(psi, v, u, 0.5 * tau), v, u


def _step_coefficients(f, lo, hi, n):
    t = math.pi * (torch.arange(4 * n, dtype=torch.float64, device="cuda") + 0.5) / (4 * n)
    fv = f(0.5 * (hi + lo) + 0.5 * (hi - lo) * torch.cos(t))
    a = torch.stack([(fv * torch.cos(k * t)).sum() for k in range(n)]) / (2 * n)
    a[0] *= 0.5
    return a.tolist()


def _gapped(e0, e1, eps, lo, hi, n):
    a, b = 0.0, 10.0
    for _ in range(200):                       # erfc(x) = 2 eps
        m = 0.5 * (a + b)
        a, b = (m, b) if math.erfc(m) > 2 * eps else (a, m)
    sigma = (e1 - e0) / (2 * a)
    mu = 0.5 * (e0 + e1)
    return _step_coefficients(lambda e: 0.5 * torch.erfc((e - mu) / sigma), lo, hi, n)


def _exp_coefficients(lo, hi, t):
    """exp(-i H t) as a Chebyshev series, to rounding."""
    R, n = 0.5 * (hi - lo), int(0.5 * (hi - lo) * abs(t)) + 60
    th = math.pi * (torch.arange(4 * n, dtype=torch.float64, device="cuda") + 0.5) / (4 * n)
    f = torch.exp(-1j * R * t * torch.cos(th))
    a = torch.stack([(f * torch.cos(k * th)).sum() for k in range(n)]) / (2 * n)
    a[0] *= 0.5
    return (a * complex(math.cos(0.5 * (hi + lo) * t), -math.sin(0.5 * (hi + lo) * t))).tolist()


def _exact_lanczos(case, seed):
    H = _Exact(case)
    v = _signs(seed, 5, 0, 0, H.N).to(torch.complex128)
    v = v / v.norm()
    vp, b, alpha, beta = torch.zeros_like(v), 0.0, [], []
    for _ in range(case["steps"]):
        w = H.apply(v[None])[0]
        a = float((v.conj() * w).real.sum())
        w = w - a * v - b * vp
        b = float(w.norm())
        alpha.append(a)
        beta.append(b)
        vp, v = v, w / b
    th, y = np.linalg.eigh(np.diag(alpha) + np.diag(beta[:-1], 1) + np.diag(beta[:-1], -1))
    pad = 0.01 * (th[-1] - th[0])
    hi = float(H.T.max() + H.v.max())          # Weyl: V_NL is attractive or absent
    lo = float(H.v.min()) if H.B is None else -math.inf
    return (max(lo, th[0] - beta[-1] * abs(y[-1, 0]) - pad),
            min(hi, th[-1] + beta[-1] * abs(y[-1, -1]) + pad))


def _exact_sigma(case, seed):
    H, p = _Exact(case), _sigma_params(case, seed)
    N, dV, L, nt = H.N, H.dV, case["neta"], case["n_tau"]
    lo, hi = p["emin"], p["emax"]
    phi = torch.from_numpy(_orbital(case, seed)).cuda()
    coef = _step_coefficients(lambda e: torch.sigmoid(-p["beta"] * (e - p["mu"])), lo, hi, p["ncoef"])
    prop = _exp_coefficients(lo, hi, p["dt"])
    ns, n_xi = case["ns"], case["n_xi"]
    nb = N // 32
    nseg = max(1, int(p["f_g"] * N / 32 + 0.5))
    amp = 1 / math.sqrt(n_xi * (32.0 * nseg / N) * dV)
    noise = torch.stack([_signs(seed, 1 if l < 0 else 2, s, max(l, 0), N)
                         for s in range(ns) for l in range(-1, L)]).reshape(ns, 1 + L, N)
    noise = noise / math.sqrt(dV)
    filt = H.series(coef, lo, hi, noise.to(torch.complex128)).real
    zb, zocc, eta = noise[:, 0], filt[:, 0], filt[:, 1:]
    pe = phi * eta
    X = -dV * (pe * H.mult(pe + 0j, H.coul).real).sum((1, 2)) / L
    psi, v, u = H.tdh(eta, H.mult(phi * zb + 0j, H.coul).real, 2.0 / L)
    tau = p["dt"] / p["m_sub"]
    idx, sgn = [], []
    for s in range(ns):
        d = torch.remainder(_shr(_words(seed, 3, s, 0, n_xi * nseg), 1) % nb * 2 +
                            (_words(seed, 3, s, 0, n_xi * nseg) & 1), nb).reshape(n_xi, nseg)
        for g in range(1, nseg):
            while True:
                hit = (d[:, :g] == d[:, g:g + 1]).any(1)
                if not bool(hit.any()):
                    break
                d[:, g] = torch.where(hit, (d[:, g] + 1) % nb, d[:, g])
        w = _words(seed, 4, s, 0, n_xi * nseg).reshape(n_xi, nseg)
        idx.append((d[:, :, None] * 32 + torch.arange(32, device="cuda")).reshape(n_xi, -1))
        sgn.append((1 - 2 * ((w[:, :, None] >> torch.arange(32, device="cuda")) & 1))
                   .reshape(n_xi, -1).double())

    def overlap(f):                            # [ns][N] -> [ns][n_xi]
        return torch.stack([amp * dV * (f[s][idx[s]] * sgn[s]).sum(1) for s in range(ns)])

    zp, zt = (zb - zocc) + 0j, zocc + 0j
    cR, dp, dm = [overlap(u)], [overlap(phi * zp)], [overlap(-phi * zt.conj())]
    for _ in range(nt):
        for _ in range(p["m_sub"]):
            psi, v, u = H.substep(psi, v, u, tau, 2.0 / L, None)
        z = H.series(prop, lo, hi, torch.stack([zp, zt]))
        zp, zt = z[0], z[1]
        cR.append(overlap(u))
        dp.append(overlap(phi * zp))
        dm.append(overlap(-phi * zt.conj()))
    nft = 1
    while nft < 4 * (nt + 1):
        nft *= 2
    F = nft * torch.fft.ifft(torch.stack(cR, -1).to(torch.complex128), n=nft, dim=-1)
    F[..., nft // 2 + 1:] = F[..., nft // 2 + 1:].conj()
    c = torch.fft.fft(F, dim=-1)[..., :nt + 1] / nft
    sp = (c * torch.stack(dp, -1)).sum(1)
    sm = (c * torch.stack(dm, -1)).sum(1)
    sig = torch.cat([sm[:, 1:].flip(1), 0.5 * (sp[:, :1] + sm[:, :1]), sp[:, 1:]], dim=1)
    return [sig.cpu().numpy(), X.cpu().numpy()]


def _exact_train(case, seed):
    x, y, mean, std = _train_inputs(case, seed)
    n = case["samples"]
    xh = (x.double() - torch.from_numpy(mean).cuda()) / torch.from_numpy(std).cuda()
    th = torch.from_numpy(systems.mlp_init(seed % 1000)).cuda()
    m, v, losses = torch.zeros_like(th), torch.zeros_like(th), []
    for t in range(1, case["steps"] + 1):
        q = th.clone().requires_grad_(True)
        W1, b1, W2, b2, w3, b3 = torch.split(q, [256 * 64, 256, 256 * 256, 256, 256, 1])
        a1 = torch.tanh(xh @ W1.view(256, 64).t() + b1)
        a2 = torch.tanh(a1 @ W2.view(256, 256).t() + b2)
        loss = ((a2 @ w3 + b3 - y.double()) ** 2).sum() / n
        g, = torch.autograd.grad(loss, q)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        th = th - 1e-3 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
        losses.append(float(loss.detach()))
    return [th.cpu().numpy(), np.array(losses)]


def exact(case, seed):
    op = case["op"]
    if op == "train":
        return _exact_train(case, seed)
    if op == "lanczos":
        return _exact_lanczos(case, seed)
    if op == "sigma":
        return _exact_sigma(case, seed)
    if op == "features":
        phi, N = _features_inputs(case, seed).double(), case["n"] ** 3
        out = []
        for s0 in range(0, case["samples"], 1024):
            m = min(1024, case["samples"] - s0)
            t = (1 << 40) | (torch.arange(s0, s0 + m, device="cuda") << 20)
            key = _sm64(_sm64(t) ^ seed)
            w = _sm64(key[:, None] + torch.arange(N // 64, device="cuda"))
            acc = torch.zeros((m, case["states"]), dtype=torch.float64, device="cuda")
            for b in range(64):
                acc += (1 - 2 * ((w >> b) & 1)).double() @ phi[:, b::64].t()
            out.append(0.5 ** 3 * acc ** 2)
        return torch.cat(out)
    H = _Exact(case)
    if op == "tdh":
        eta, dv = _tdh_inputs(case, seed)
        w = 2.0 / case["neta"]
        psi, v, u = H.tdh(eta.double(), dv.double(), w)
        K = H.kb_exponential(0.5 * case["dt"]) if H.B is not None else None
        for _ in range(case["nsub"]):
            psi, v, u = H.substep(psi, v, u, case["dt"], w, K)
        return [psi, v, u]
    g = _gen(seed)
    if op == "filter":
        x = _noise(g, case["nvec"], H.N, H.dV)
        if case["prec"] == "c128":
            x = x.to(torch.complex128)
        coef = _gapped(*_gap(case), 1e-7, *_interval(case), case["terms"])
        return H.series(coef, *_interval(case), x.to(torch.complex128))
    x = torch.randn((case["nvec"], H.N), generator=g, device="cuda",
                    dtype=torch.complex64).to(torch.complex128)
    if op == "hpsi":
        return H.apply(x)
    coef = _exp_coefficients(*_interval(case), case["dt"])
    for _ in range(case["steps"]):
        x = H.series(coef, *_interval(case), x)
    return x
