"""The work that users have this framework do, as cases that can be timed and checked.

A case is one stretch of a simulation through the public binding: some steps
with their samples, then the read-out that ends the stretch.  ``listed``
gives the fixed cases, ``draw`` others of the same ranges, ``exact`` the same
stretch in plain FP64 torch.
"""
import math

import numpy as np
import torch

import paper_1202_4748_amd as lbf

# Ginzburg-Landau parameters of the repository's workloads: the critical
# point search around a = 0 (the verification run takes a = 0.05, b = 0)
CRITICAL = dict(a=0.0, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=1.0, init_sigma=1e-3)
SWEEP_L = (8, 12, 16, 24, 32, 48)
SWEEP_A = (-0.02, -0.02 / 3, 0.02 / 3, 0.02)


def _case(**kw):
    c = dict(model="force", L=16, replicas=1, a=0.0, b=0.1, tau=1.0, storage="fp32", steps=100, sample_every=10,
             sk3_stride=0, hist_bins=0, sweep=False, resume=False, rho=False, j=False, f=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest lattice of the workloads, to be looked at after a short
        # run: launches and latency count
        _case(name="force_16", L=16, steps=200, j=True, rho=True, f=True),
        # a lattice edge that no tile divides and that is no multiple of four
        _case(name="force_50", L=50, steps=100, rho=True, j=True),
        # the verification run: Gaussian statics with the 3D structure factor
        _case(name="verify_64", L=64, a=0.05, b=0.0, steps=200, sk3_stride=2, rho=True),
        # half-precision storage on a middling lattice, with the histograms of
        # the order parameter
        _case(name="fp16_96", L=96, storage="fp16", steps=100, hist_bins=64, rho=True),
        # the plain throughput run and its density field at the end
        _case(name="force_256", L=256, steps=100, rho=True),
        # the precision variant: the largest lattice, FP16 storage
        _case(name="fp16_512", L=512, storage="fp16", steps=20),
        # the finite-size sweep: 96 replicas of six lattice edges in one handle
        _case(name="sweep_96", L=48, replicas=96, sweep=True, steps=400),
        # the paper's own model on D3Q19
        _case(name="eq_256", model="eq", L=256, steps=100, rho=True),
        # the paper's lattice, one realization, to its spectra
        _case(name="d2q9_256", model="d2q9", L=256, steps=500, rho=True, j=True),
        # the largest two-dimensional lattice
        _case(name="d2q9_2048", model="d2q9", L=2048, steps=400),
        # many realizations of the paper's lattice side by side
        _case(name="d2q9_256_x64", model="d2q9", L=256, replicas=64, steps=500),
        # resume from a stored state, go on for a little, store the state again
        _case(name="resume_64", L=64, steps=20, sample_every=0, resume=True, rho=True, j=True, f=True),
    ]


def draw(rng):
    """One more case: any model, lattice edges over their whole range (odd
    ones among them), with the samples and read-outs the listed ones have."""
    kind = rng.choice(("force", "force", "fp16", "eq", "d2q9", "d2q9", "d2q9_batch", "batch", "resume"))
    # around the critical point, or the Gaussian fluid
    a, b = (round(rng.uniform(-0.02, 0.05), 4), 0.1) if rng.random() < 0.7 else (round(rng.uniform(0.02, 0.06), 4), 0.0)
    tau = round(rng.uniform(0.7, 1.1), 2)
    if kind in ("eq", "d2q9", "d2q9_batch"):
        a = abs(a)  # below the critical point these models' c_s^2 turns negative

    def edge(lo, hi):
        L = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        k = rng.choice((1, 2, 4, 8, 16))  # ragged edges as well as those with block levels
        return max(lo, L // k * k)

    def steps(sites, most):
        n = min(most, int(1.5e9 // sites))
        return max(20, n // 10 * 10)

    if kind == "d2q9":
        L = edge(32, 2048)
        if L > 512 and L & (L - 1):  # direct transforms on large edges take seconds
            L = 1 << (L.bit_length() - 1)
        big = L > 1024
        return _case(model="d2q9", L=L, a=a, b=b, tau=tau, steps=400 if big else steps(L * L * 4, 500), rho=not big,
                     j=not big)
    if kind == "d2q9_batch":
        L, R = edge(24, 256), rng.randint(2, 64)
        return _case(model="d2q9", L=L, replicas=R, a=a, b=b, tau=tau, steps=200)
    if kind == "batch":
        L, R = edge(8, 48), rng.randint(2, 64)
        return _case(L=L, replicas=R, a=a, b=b, tau=tau, steps=100)
    if kind == "resume":
        L = edge(8, 72)
        return _case(L=L, a=a, b=b, tau=tau, steps=20, sample_every=0, resume=True, rho=True, j=True, f=True)
    L = edge(8, 256)
    n = steps(L ** 3, 200)
    if kind == "eq":
        return _case(model="eq", L=L, a=a, b=b, tau=tau, steps=n, rho=True)
    if kind == "fp16":
        return _case(L=L, a=a, b=b, tau=tau, storage="fp16", steps=n, hist_bins=rng.choice((0, 64)), rho=True)
    return _case(L=L, a=a, b=b, tau=tau, steps=n, sk3_stride=rng.choice((0, 0, 2)) if L <= 64 else 0, rho=True)


# --------------------------------------------------------------------------
# what a user's program holds, and one stretch of it
# --------------------------------------------------------------------------
def _params(c):
    p = dict(CRITICAL, a=c["a"], b=c["b"], tau=c["tau"])
    if c["model"] != "d2q9":
        p.update(storage=c["storage"], sample_every=c["sample_every"], sk3_stride=c["sk3_stride"],
                 hist_bins=c["hist_bins"], hist_range=0.2 if c["hist_bins"] else 0.0,
                 series_capacity=64 if c["sample_every"] else 0)
        if c["model"] == "eq":
            p["eq_pressure"] = True
    else:
        p["sample_every"] = c["sample_every"]
    return p


def _replicas(c, seed):
    """Lattice edges, coefficients a and seeds of the replicas."""
    if c["sweep"]:
        per = c["replicas"] // (len(SWEEP_L) * len(SWEEP_A))
        Ls = [L for L in SWEEP_L for _ in range(len(SWEEP_A) * per)]
        As = [a for _ in SWEEP_L for a in SWEEP_A for _ in range(per)]
    else:
        Ls, As = [c["L"]] * c["replicas"], [c["a"]] * c["replicas"]
    return Ls, As, [1000 * seed + 7 * r for r in range(c["replicas"])]


def _stored_state(c, seed):
    """A stored state to resume from, f[19][L^3]: a fluctuating density and
    momentum with some non-equilibrium part on every population."""
    rng = np.random.default_rng(seed)
    N = c["L"] ** 3
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    f = w[:, None] * (1.0 + 0.02 * rng.standard_normal(N)[None, :] + 0.01 * rng.standard_normal((19, N)))
    odd = 0.06 * rng.standard_normal((9, N))
    f[1::2] += w[1::2, None] * odd
    f[2::2] -= w[2::2, None] * odd
    return f


def prepare(case, seed):
    c = dict(case)
    Ls, As, seeds = _replicas(c, seed)
    p = _params(c)
    if c["model"] == "d2q9":
        if c["replicas"] == 1:
            sim = lbf.Sim2D(c["L"], seeds[0], **p)
        else:
            sim = lbf.Sim2D.batch(c["L"], seeds, [p] * c["replicas"])
    elif c["replicas"] == 1:
        sim = lbf.Sim(c["L"], seeds[0], **p)
    else:
        sim = lbf.Sim.batch(Ls, seeds, [dict(p, a=a) for a in As])
    sim.sync()
    return {"case": c, "sim": sim, "Ls": Ls, "stored": _stored_state(c, seed) if c["resume"] else None}


_LEVEL_KEYS = ("m", "m2", "m3", "m4", "abs_m", "E", "E2")


def _moments(sim, r):
    m = sim.moments(r, series=True)
    return {"n_samples": m["n_samples"], "mass": m["mass"], "momentum": m["momentum"], "sk": m["sk"],
            "levels": np.array([[lv[k] for k in _LEVEL_KEYS] for lv in m["levels"]]).reshape(-1, 7),
            "series": m["series"]}


def _stack(ms, Ls):
    """The replicas' moments, those of one lattice edge in one array."""
    out = {}
    for L in sorted(set(Ls)):
        mine = [m for m, l in zip(ms, Ls) if l == L]
        out[str(L)] = {k: np.stack([np.asarray(m[k]) for m in mine]) for k in mine[0]}
    return out


def run(state):
    c, sim = state["case"], state["sim"]
    if c["resume"]:
        sim.set_populations(state["stored"])
        sim.set_step(1000)
    sim.step(c["steps"])
    out = {}
    if c["model"] == "d2q9":
        spectra = [sim.spectra(r) for r in range(c["replicas"])]
        if c["replicas"] == 1:
            out.update(spectra[0])
        else:
            out.update({k: [s[k] for s in spectra] if k == "n_samples" else np.stack([s[k] for s in spectra])
                        for k in spectra[0]})
            out["n_samples"] = np.array(out["n_samples"])
        if c["rho"]:
            out.update(sim.fields())
        return out
    if c["replicas"] > 1:
        return _stack([_moments(sim, r) for r in range(c["replicas"])], state["Ls"])
    if c["sample_every"]:
        out.update(_moments(sim, 0))
    if c["hist_bins"]:
        out["counts"] = sim.histogram().astype(np.int64)
    if c["sk3_stride"]:
        s = sim.sk3()
        out.update(sk3_samples=s["n_samples"], sk3_sum=s["sum_C"])
    if c["rho"]:
        out.update(sim.fields(rho=c["rho"], j=c["j"], f=c["f"]))
    return out


def work(case):
    """Per step every population read and written once, in its storage
    format; about 700 (D3Q19) and 300 (D2Q9) operations a site and step."""
    c = dict(case)
    if c["model"] == "d2q9":
        sites, q, ops = c["replicas"] * c["L"] ** 2, 9, 300
    else:
        sites, q, ops = sum(L ** 3 for L in _replicas(c, 0)[0]), 19, 700
    size = 2 if c["storage"] == "fp16" else 4
    return {"bytes": 2.0 * q * size * sites * c["steps"], "flops": float(ops) * sites * c["steps"]}


# --------------------------------------------------------------------------
# the same stretch in FP64 torch
# --------------------------------------------------------------------------
C3 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
      (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1),
      (0, -1, 1)]
W3 = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
C2 = [(0, 0), (1, 0), (-1, 0), (0, 1), (0, -1), (1, 1), (-1, -1), (1, -1), (-1, 1)]
W2 = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4


def _basis3():
    rows = []
    for x, y, z in C3:
        s = x * x + y * y + z * z
        rows.append([1, x, y, z, s - 1, 3 * x * x - s, y * y - z * z, x * y, y * z, z * x, (3 * s - 5) * x,
                     (3 * s - 5) * y, (3 * s - 5) * z, (y * y - z * z) * x, (z * z - x * x) * y, (x * x - y * y) * z,
                     3 * s * s - 6 * s + 1, (2 * s - 3) * (3 * x * x - s), (2 * s - 3) * (y * y - z * z)])
    return np.array(rows, dtype=float).T


def _basis2():
    rows = []
    for x, y in C2:
        s = x * x + y * y
        rows.append([1, x, y, 3 * s - 2, x * x - y * y, x * y, (3 * s - 4) * x, (3 * s - 4) * y,
                     9 * s * s - 15 * s + 2])
    return np.array(rows, dtype=float).T


def _philox(site, t, call, seeds):
    """Philox4x32-10 words of counters (site, t_lo, call, t_hi), one key per replica."""
    M = 0xFFFFFFFF
    k0 = torch.tensor([s & M for s in seeds], device=site.device).view(-1, 1)
    k1 = torch.tensor([s >> 32 & M for s in seeds], device=site.device).view(-1, 1)
    zero = torch.zeros((len(seeds), 1), dtype=torch.int64, device=site.device)
    c0, c1, c2, c3 = site.view(1, -1) + zero, zero + (t & M), zero + call, zero + (t >> 32)
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c2 = ((p1 >> 32) & M) ^ c1 ^ k0, ((p0 >> 32) & M) ^ c3 ^ k1
        c1, c3 = p1 & M, p0 & M
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c0, c1, c2, c3


def _normals(site, t, call, seeds):
    u = [((w >> 9).double() + 0.5) * 2.0 ** -23 for w in _philox(site, t, call, seeds)]
    r0, r1 = torch.sqrt(-2 * torch.log(u[0])), torch.sqrt(-2 * torch.log(u[2]))
    a0, a1 = 2 * math.pi * u[1], 2 * math.pi * u[3]
    return r0 * torch.cos(a0), r0 * torch.sin(a0), r1 * torch.cos(a1), r1 * torch.sin(a1)


def _shift(v, c):
    """v(x + c) on the periodic lattice, axes [replica, (z,) y, x]."""
    return torch.roll(v, shifts=tuple(-k for k in c), dims=tuple(range(v.dim() - 1, v.dim() - 1 - len(c), -1)))


class _Fluid:
    """Replicas of one lattice edge: f, a list of [R, (L,) L, L] arrays."""

    def __init__(self, c, L, a, seeds, dev):
        self.L, self.seeds, self.dev, self.model = L, seeds, dev, c["model"]
        self.dim = 2 if self.model == "d2q9" else 3
        self.C, self.W = (C2, W2) if self.dim == 2 else (C3, W3)
        self.E = torch.tensor(_basis2() if self.dim == 2 else _basis3(), device=dev)
        self.N = (self.E ** 2) @ torch.tensor(self.W, dtype=torch.float64, device=dev)
        self.B = torch.tensor(self.W, device=dev, dtype=torch.float64)[:, None] * (self.E / self.N[:, None]).T
        self.R, self.t = len(seeds), 0
        p = CRITICAL
        self.b, self.kappa, self.rho_c, self.kT, self.tau = c["b"], p["kappa"], p["rho_c"], p["kT"], c["tau"]
        self.a = torch.tensor(a, dtype=torch.float64, device=dev).view(-1, 1)
        self.shape = (self.R,) + (L,) * self.dim
        n = L ** self.dim
        rho = torch.empty((self.R, n), dtype=torch.float64, device=dev)
        for lo, hi in self.chunks():
            site = torch.arange(lo, hi, device=dev)
            rho[:, lo:hi] = p["rho_c"] + p["init_sigma"] * _normals(site, 0, 1 << 16, seeds)[0]
        if self.model == "d2q9":  # the equilibrium of that density at rest
            d, g, lap = self.derivatives((rho - self.rho_c).view(self.shape))
            m = [d + self.rho_c, 0 * d, 0 * d] + self.equilibrium2(d, [0 * d, 0 * d], g, lap)
            self.f = [sum(self.B[q, k] * m[k] for k in range(9)).view(self.shape) for q in range(9)]
        else:
            self.f = [(w * rho).view(self.shape) for w in self.W]

    def chunks(self):
        """Site ranges that keep the temporaries small."""
        n = self.L ** self.dim
        size = max(1, (1 << 22) // self.R)
        return [(lo, min(n, lo + size)) for lo in range(0, n, size)]

    def derivatives(self, d):
        """Density deviation, gradient and Laplacian, flattened to [R, sites]."""
        g, lap = [0.0] * self.dim, 0.0
        for c, w in zip(self.C[1:], self.W[1:]):
            v = _shift(d, c)
            lap = lap + 6 * w * (v - d)
            for k in range(self.dim):
                if c[k]:
                    g[k] = g[k] + 3 * w * c[k] * v
        flat = (self.R, -1)
        return d.reshape(flat), [x.reshape(flat) for x in g], lap.reshape(flat)

    def pressure(self, d, a):
        f0 = a / 2 * d ** 2 + self.b / 4 * d ** 4
        rho = self.rho_c + d
        return rho * (a * d + self.b * d ** 3) - f0, rho * (a + 3 * self.b * d ** 2)

    def stress(self, d, u, g, lap):
        """The equilibrium's second moment, and its isotropic part."""
        nu, rho, k = (self.tau - 0.5) / 3, self.rho_c + d, self.kappa
        p0, _ = self.pressure(d, self.a)
        iso = p0 - k * rho * lap - k / 2 * sum(x * x for x in g)
        ug = sum(x * y for x, y in zip(u, g))

        def P(i, j):
            return (k * g[i] * g[j] + rho * u[i] * u[j] + nu * (u[i] * g[j] + u[j] * g[i]) +
                    (iso + nu * ug if i == j else 0.0))
        return P, iso

    def equilibrium2(self, d, u, g, lap):
        P, _ = self.stress(d, u, g, lap)
        rho, p0 = self.rho_c + d, self.pressure(d, self.a)[0]
        xx, yy = P(0, 0), P(1, 1)
        return [3 * (xx + yy) - 2 * rho, xx - yy, P(0, 1), 0 * d, 0 * d,
                2 * rho - 6 * (p0 - self.kappa * rho * lap) - 3 * self.kappa * sum(x * x for x in g)]

    def step(self):
        R, flat = self.R, (self.R, -1)
        d_field = sum(self.f) - self.rho_c
        out = [torch.empty_like(x).view(flat) for x in self.f]
        f = [x.reshape(flat) for x in self.f]
        if self.model == "force":
            d, _, lap = self.derivatives(d_field)
            mu = self.a * d + self.b * d ** 3 - self.kappa * lap
            gmu, grho = self.derivatives(mu.view(self.shape))[1], self.derivatives(d_field)[1]
            del lap, mu
        else:
            d, grho, lap_all = self.derivatives(d_field)
        gam = 1 - 1 / self.tau
        N = [float(x) for x in self.N]
        for lo, hi in self.chunks():
            cut = slice(lo, hi)
            site = torch.arange(lo, hi, device=self.dev)
            m = torch.matmul(self.E, torch.stack([x[:, cut] for x in f]).reshape(len(f), -1)).view(len(f), R, -1)
            m = list(m)
            rho, dd = m[0], m[0] - self.rho_c
            if self.model == "force":
                F = [-rho * gm[:, cut] + gr[:, cut] / 3 for gm, gr in zip(gmu, grho)]
                u = [(m[1 + k] + F[k] / 2) / rho for k in range(3)]
                u2, uF = sum(x * x for x in u), sum(x * y for x, y in zip(u, F))
                eq = {4: rho * u2, 5: rho * (3 * u[0] ** 2 - u2), 6: rho * (u[1] ** 2 - u[2] ** 2),
                      7: rho * u[0] * u[1], 8: rho * u[1] * u[2], 9: rho * u[2] * u[0]}
                src = {4: 2 * uF, 5: 2 * (3 * u[0] * F[0] - uF), 6: 2 * (u[1] * F[1] - u[2] * F[2]),
                       7: u[0] * F[1] + u[1] * F[0], 8: u[1] * F[2] + u[2] * F[1], 9: u[2] * F[0] + u[0] * F[2]}
                for k in range(3):
                    m[1 + k] = m[1 + k] + F[k]
                for k in range(4, 19):
                    m[k] = gam * m[k] + ((1 - gam) * eq[k] + (1 + gam) / 2 * src[k] if k < 10 else 0.0)
                sig = torch.sqrt(3 * rho * self.kT * (1 - gam ** 2))
                for call in range(4):
                    for k, g in enumerate(_normals(site, self.t, call, self.seeds)):
                        if 4 * call + k < 15:
                            m[4 + 4 * call + k] += sig * math.sqrt(N[4 + 4 * call + k]) * g
            else:
                g, lap = [x[:, cut] for x in grho], lap_all[:, cut]
                u = [m[1 + k] / rho for k in range(self.dim)]
                cs2 = self.pressure(dd, self.a)[1]
                sig = torch.sqrt(3 * rho * self.kT * (1 - gam ** 2))
                if self.dim == 2:
                    eq = self.equilibrium2(dd, u, g, lap)
                    for k in range(3, 9):
                        m[k] = eq[k - 3] + gam * (m[k] - eq[k - 3])
                    n = _normals(site, self.t, 0, self.seeds) + _normals(site, self.t, 1, self.seeds)[:2]
                    l33 = torch.sqrt(4 * (2 - 3 * cs2))
                    l83 = 12 * (cs2 - 1 / 3) / l33
                    l88 = torch.sqrt(16 * (1.25 - 0.75 * cs2) - l83 ** 2)
                    m[3] = m[3] + sig * l33 * n[0]
                    for k in range(4, 8):
                        m[k] = m[k] + sig * math.sqrt(N[k]) * n[k - 3]
                    m[8] = m[8] + sig * (l83 * n[0] + l88 * n[5])
                else:
                    P, iso = self.stress(dd, u, g, lap)
                    xx, yy, zz = P(0, 0), P(1, 1), P(2, 2)
                    eq = {4: xx + yy + zz - rho, 5: 2 * xx - yy - zz, 6: yy - zz, 7: P(0, 1), 8: P(1, 2), 9: P(2, 0),
                          16: rho - 3 * iso}
                    n = [x for call in range(4) for x in _normals(site, self.t, call, self.seeds)]
                    l44 = torch.sqrt(5 / 3 - 3 * cs2)
                    l164 = (3 * cs2 - 1) / l44
                    l1616 = torch.sqrt(3 - 3 * cs2 - l164 ** 2)
                    for k in range(4, 19):
                        m[k] = gam * m[k] + (1 - gam) * eq.get(k, 0.0)
                        if k not in (4, 16):
                            m[k] = m[k] + sig * math.sqrt(N[k]) * n[k - 4]
                    m[4] = m[4] + sig * l44 * n[0]
                    m[16] = m[16] + sig * (l164 * n[0] + l1616 * n[12])
            new = torch.matmul(self.B, torch.stack(m).reshape(len(m), -1)).view(len(m), R, -1)
            for q in range(len(m)):
                out[q][:, cut] = new[q]
        self.f = [_shift(x.view(self.shape), tuple(-k for k in c)) for x, c in zip(out, self.C)]
        self.t += 1

    def fields(self):
        f = torch.stack([x[0].reshape(-1) for x in self.f])
        C = torch.tensor(self.C, dtype=torch.float64, device=self.dev)
        return f.sum(0), C.T @ f, f


def _levels(L):
    out = []
    while L % 2 == 0 and L > 1:
        L //= 2
        out.append(L)
    return out


class _Samples3:
    """Accumulated observables of the three-dimensional models."""

    def __init__(self, fl, c):
        self.fl, self.c, self.n = fl, c, 0
        self.levels, self.sk, self.series, self.sk3 = 0.0, 0.0, [], 0.0
        self.n3 = 0

    def take(self):
        fl, L, R = self.fl, self.fl.L, self.fl.R
        d = sum(fl.f) - fl.rho_c
        dbar = d.mean(dim=(1, 2, 3)).view(-1, 1, 1, 1)
        rho0 = fl.rho_c + dbar
        phi = (d - dbar) / rho0
        lev = []
        for Lb in _levels(L):
            n = L // Lb

            def boxes(v):
                return v.reshape(R, n, Lb, n, Lb, n, Lb).sum(dim=(2, 4, 6)).reshape(R, -1)
            m, e = boxes(phi) / Lb ** 3, boxes(phi * phi) / (2 * Lb ** 3)
            lev.append(torch.stack([m.sum(1), (m ** 2).sum(1), (m ** 3).sum(1), (m ** 4).sum(1), m.abs().sum(1),
                                    e.sum(1), (e ** 2).sum(1)], dim=1) / n ** 3)
        lev = torch.stack(lev, dim=1) if lev else torch.zeros((R, 0, 7), dtype=torch.float64, device=fl.dev)
        count = torch.tensor([(L // Lb) ** 3 for Lb in _levels(L)], dtype=torch.float64, device=fl.dev).view(1, -1, 1)
        self.levels = self.levels + lev * count
        sk = []
        for axis in (3, 2, 1):  # x, y, z
            plane = phi.sum(dim=[k for k in (1, 2, 3) if k != axis])
            sk.append((torch.fft.fft(plane, dim=1).abs() ** 2 / L ** 3)[:, 1:max(L // 2, 1)])
        self.sk = self.sk + torch.stack(sk, dim=1)
        mom = [sum(x * c[k] for x, c in zip([y.sum(dim=(1, 2, 3)) for y in fl.f], fl.C)) for k in range(3)]
        head = torch.stack([torch.full((R,), float(fl.t), dtype=torch.float64, device=fl.dev),
                            sum(y.sum(dim=(1, 2, 3)) for y in fl.f)] + mom, dim=1)
        self.series.append(torch.cat([head, lev.reshape(R, -1)], dim=1))
        self.n += 1
        c = self.c
        if c["sk3_stride"] and fl.t % (c["sample_every"] * c["sk3_stride"]) == 0:
            C = torch.fft.fftn(phi[0]).abs() ** 2 / L ** 3
            k = torch.fft.fftfreq(L, 1.0 / L, device=fl.dev, dtype=torch.float64)
            r = torch.sqrt(k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2)
            s = torch.floor(r + 0.5).long().reshape(-1)
            w = C.reshape(-1).clone()
            w[s == 0] = 0.0
            self.sk3 = self.sk3 + torch.bincount(s, weights=w)
            self.n3 += 1

    def result(self):
        fl = self.fl
        return {"n_samples": np.full(fl.R, self.n), "mass": sum(y.sum(dim=(1, 2, 3)) for y in fl.f).cpu().numpy(),
                "momentum": None, "sk": self.sk.cpu().numpy(), "levels": self.levels.cpu().numpy(),
                "series": torch.stack(self.series, dim=1)[:, -64:].cpu().numpy()}


def _spectra2(fl, acc):
    L = fl.L
    v = [sum(fl.f)] + [sum(x * c[k] for x, c in zip(fl.f, fl.C)) for k in range(2)]
    v[0] = v[0] - fl.rho_c
    r, jx, jy = (torch.fft.fft2(x) for x in v)
    m = torch.fft.fftfreq(L, 1.0 / L, device=fl.dev, dtype=torch.float64)
    if L % 2 == 0:
        m[L // 2] = L // 2
    kn = torch.sqrt(m[:, None] ** 2 + m[None, :] ** 2)
    kn[0, 0] = 1.0
    hx, hy = m[None, :] / kn, m[:, None] / kn
    add = {"S": r, "Jx": jx, "Jy": jy, "Jpar": hx * jx + hy * jy, "Jperp": hx * jy - hy * jx}
    for k, x in add.items():
        acc[k] = acc.get(k, 0.0) + x.abs() ** 2 / L ** 2


def exact(case, seed):
    c = dict(case)
    Ls, As, seeds = _replicas(c, seed)
    sites = sum(L ** (2 if c["model"] == "d2q9" else 3) for L in Ls)
    if sites * c["steps"] > 3.0e9:
        return None  # minutes in FP64
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    found = {}
    for L in sorted(set(Ls)):
        mine = [r for r, l in enumerate(Ls) if l == L]
        fl = _Fluid(c, L, [As[r] for r in mine], [seeds[r] for r in mine], dev)
        if c["resume"]:
            fl.f = [torch.from_numpy(x).to(dev).view(fl.shape) for x in _stored_state(c, seed)]
            fl.t = 1000
        s, acc = _Samples3(fl, c), {}
        for _ in range(c["steps"]):
            fl.step()
            if c["sample_every"] and fl.t % c["sample_every"] == 0:
                if c["model"] == "d2q9":
                    _spectra2(fl, acc)
                else:
                    s.take()
        if c["model"] == "d2q9":
            one = c["replicas"] == 1
            out = {k: (v[0] if one else v).cpu().numpy() for k, v in acc.items()}
            n = c["steps"] // c["sample_every"]
            out["n_samples"] = n if one else np.full(c["replicas"], n)
            if c["rho"]:
                rho, j, _ = fl.fields()
                out.update(rho=rho.cpu().numpy(), j=j.cpu().numpy())
            return out
        found[str(L)] = s.result() if c["sample_every"] else {}
    if c["replicas"] > 1:
        return found
    out = {k: None if v is None else v[0] for k, v in found[str(c["L"])].items()}
    if "mass" in out:
        out.update(mass=float(out["mass"]), n_samples=int(out["n_samples"]))
    if c["hist_bins"]:
        out["counts"] = None  # a box value next to a bin's edge may be counted on either side
    if c["sk3_stride"]:
        out.update(sk3_samples=s.n3, sk3_sum=s.sk3.cpu().numpy())
    if c["rho"]:
        rho, j, f = fl.fields()
        got = {"rho": rho, "j": j, "f": f}
        out.update({k: v.cpu().numpy() for k, v in got.items() if c[k]})
    return out
