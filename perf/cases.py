"""Performance cases: the calls a program built on this library spends its time in.

Every case is a dict of plain values.  `prepare` makes what such a program has
in hand (a context, particles, network weights), `run` is one pass through the
public entry points, `exact` the same outputs in 64-bit torch and numpy
(cosmology, initial conditions, particle-mesh step, network and their
derivatives written out here), `work` the bytes and operations a pass cannot
do without.

Kinds:
  run          a sorted simulation restarted from a snapshot: `calls` pm_step
               calls, then the particles back in lattice order (displacement
               since the snapshot, momentum)
  learned      the same with pm_learned_step and the trained correction
  train        one training step of the correction: loss, gradient, Adam
  reconstruct  one iteration of the initial-mode reconstruction: initial
               conditions, steps, density and the reverse mode of all of them
  reverse      one unsorted step and its reverse mode
  force        forces at given positions (the target of a training pair)
  ic           initial conditions from white noise
  power        the total power spectrum and the CDM x neutrino cross spectrum
"""
import math
import os

import numpy as np
import torch

from paper_2007_13394_amd import diff, inputs, learn, pm

DEV = "cuda"
THETA = os.path.join(os.path.dirname(os.path.abspath(learn.__file__)), "c4_learned_theta.npy")
COSMO = dict(omega_m=0.3, h=0.7, n_s=0.96, sigma8=0.8, T_cmb=2.7255, N_eff=3.046)


# ---------------------------------------------------------------- the cases
def listed():
    def case(name, kind, mesh, cdm, sites, box, m_nu=0.1, a=0.5, calls=1, steps=10, shell=10, fib=3, bins=0):
        return dict(name=name, kind=kind, mesh=mesh, cdm=cdm, sites=sites, shell=shell, fib=fib, box=float(box),
                    m_nu=m_nu, a=a, calls=calls, steps=steps, bins=bins)
    return [
        # a small whole run (test runs, ensembles of tiny boxes): launches and latency
        case("run-64", "run", 64, 32, 8, 256, a=0.3, calls=11),
        # a whole ten-step run of 2.4 M particles
        case("run-256", "run", 256, 128, 16, 256, a=0.3, calls=11),
        # the middle of a 25-step production run, 19 M particles, two cells per CDM particle
        case("run-512", "run", 512, 256, 32, 512, m_nu=0.2, a=0.5, calls=4, steps=12),
        # the fine-mesh truth of the learned correction: four cells per particle, the mesh dominates
        case("run-1024", "run", 1024, 256, 32, 256, a=0.5, calls=3, steps=12),
        # the learned correction in use: one cell per particle, the network and the particles dominate
        case("learned-256", "learned", 256, 256, 32, 256, a=0.5, calls=3, steps=12),
        # training it, on the small instance and at full size
        case("train-64", "train", 64, 64, 8, 256, a=0.5),
        case("train-256", "train", 256, 256, 32, 256, a=0.5),
        # reconstruction of the initial modes: a whole iteration of a small box
        case("reconstruct-64", "reconstruct", 64, 32, 8, 256, calls=2),
        # one link of the chain at the size of a reconstruction run
        case("reverse-256", "reverse", 256, 128, 16, 256, a=0.5),
        # forces for training pairs, from an unsorted context
        case("force-512", "force", 512, 256, 32, 512, m_nu=0.2, a=0.5),
        # initial conditions of the 19 M particle run
        case("ic-512", "ic", 512, 256, 32, 512, m_nu=0.2, a=0.01),
        # spectra of its snapshot
        case("power-512", "power", 512, 256, 32, 512, m_nu=0.2, a=0.5, bins=256),
    ]


def draw(rng):
    kind = rng.choice(["run", "run", "learned", "train", "reconstruct", "reverse", "force", "ic", "power"])
    top = {"run": 9, "learned": 8, "train": 7, "reconstruct": 7, "reverse": 8, "force": 9, "ic": 9, "power": 9}[kind]
    mesh = 1 << rng.randint(4 if kind in ("train", "reverse", "force") else 5, top)
    cdm = max(8, mesh >> rng.choice([0, 1, 1, 2]))
    if cdm > 256:
        cdm = 256
    # ragged neutrino segments: any shell and direction counts, down to a single site
    sites = max(1, cdm >> rng.choice([2, 3, 3, 4]))
    shell, fib = rng.randint(1, 12), rng.randint(0, 5)
    while sites ** 3 * shell * (2 * fib + 1) > 6_000_000:
        sites //= 2
    return dict(kind=kind, mesh=mesh, cdm=cdm, sites=sites, shell=shell, fib=fib, box=rng.choice([200.0, 256.0, 500.0]),
                m_nu=round(rng.uniform(0.06, 0.3), 3), a=0.01 if kind == "ic" else round(rng.uniform(0.3, 0.6), 3),
                calls=rng.randint(1, 4) if kind in ("run", "learned") else rng.randint(1, 3), steps=rng.randint(8, 25),
                bins=rng.randint(8, mesh) if kind == "power" else 0)


def _config(case):
    return inputs.config("C1", box=case["box"], n_mesh=case["mesh"], n_cdm=case["cdm"], n_sites=case["sites"],
                         n_shell=case["shell"], n_fib=case["fib"], m_nu=(case["m_nu"] / 3,) * 3,
                         a0=case["a"] if case["kind"] == "ic" else 0.05)


def _count(case):
    return case["cdm"] ** 3 + case["sites"] ** 3 * case["shell"] * (2 * case["fib"] + 1)


def _calls(case):
    """(a_force, a_kick0, a_kick1, a_drift1) of the first `calls` calls of a
    run of `steps` steps uniform in a from the start to today."""
    n, a0 = case["steps"], (0.05 if case["kind"] == "reconstruct" else case["a"])
    a = [a0 + (1.0 - a0) * i / n for i in range(n)] + [1.0]
    half = [0.5 * (a[i] + a[i + 1]) for i in range(n)]
    calls = [(a[i], a[0] if i == 0 else half[i - 1], half[i] if i < n else a[n], a[min(i + 1, n)])
             for i in range(n + 1)]
    return calls[:case["calls"]]


# ---------------------------------------------------------------- inputs
def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _displacement(nc, mesh, rms, gen):
    """A Gaussian displacement field on the CDM lattice (mesh cells, given rms
    per axis): the gradient of a potential with a red spectrum."""
    w = torch.fft.rfftn(torch.randn((nc,) * 3, generator=gen, device=DEV, dtype=torch.float32))
    k = [torch.fft.fftfreq(nc, device=DEV) * nc, torch.fft.fftfreq(nc, device=DEV) * nc,
         torch.fft.rfftfreq(nc, device=DEV) * nc]
    k = [k[0][:, None, None], k[1][None, :, None], k[2][None, None, :]]
    kk = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    kk[0, 0, 0] = 1.0
    w = w * kk ** -1.5 * torch.exp(-kk / (0.35 * nc) ** 2)
    s = torch.stack([torch.fft.irfftn(1j * k[d] * w, s=(nc,) * 3).reshape(-1) for d in range(3)])
    return s * (rms / s.std())


def _wrap(x, n):
    x = torch.remainder(x, float(n))
    x[x >= n] = 0.0
    return x


def _snapshot(case, seed):
    """Particles of an evolved run, float32 [3, P]: CDM on the displaced
    lattice with a tenth of it in clumps, neutrinos spread out with thermal
    momenta; and the linear force of the displacement field."""
    gen, nc, n = _generator(seed), case["cdm"], case["mesh"]
    c = nc ** 3
    i = torch.arange(c, device=DEV)
    q = torch.stack([i // nc ** 2, i // nc % nc, i % nc]).float() * (n / nc)
    s = _displacement(nc, n, (0.1 + 2.0 * case["a"]) * n / nc * 0.8, gen)
    x = q + s
    clump = torch.randint(0, c, (c // 10,), generator=gen, device=DEV)
    centre = torch.rand((3, c // 2000 + 1), generator=gen, device=DEV) * n
    pick = torch.randint(0, centre.shape[1], (c // 10,), generator=gen, device=DEV)
    # one place per particle also where `clump` names it twice
    where = torch.full((c,), -1, device=DEV, dtype=torch.int64).scatter_reduce_(0, clump, pick, "amax")
    near = centre[:, where.clamp(min=0)] + 0.7 * torch.randn((3, c), generator=gen, device=DEV)
    x = torch.where(where >= 0, near, x)
    p = case["a"] ** 1.5 * s + 0.05 * torch.randn((3, c), generator=gen, device=DEV)
    f = 1.5 * COSMO["omega_m"] * s
    nu = _count(case) - c
    xn = torch.rand((3, nu), generator=gen, device=DEV) * n
    pn = torch.randn((3, nu), generator=gen, device=DEV) * (8.0 * n / case["box"])
    fn = 0.2 * torch.randn((3, nu), generator=gen, device=DEV)
    return (_wrap(torch.cat([x, xn], 1), n).contiguous(), torch.cat([p, pn], 1).contiguous(),
            torch.cat([f, fn], 1).contiguous())


def _theta(seed):
    """The trained correction, one per cent off (a point on a training path)."""
    theta = learn.load_params(THETA, DEV)
    return theta * (1.0 + 0.01 * torch.randn(theta.shape, generator=_generator(seed + 77), device=DEV))


def _white(case, seed):
    return torch.randn((case["cdm"],) * 3, generator=_generator(seed), device=DEV)


def _pool_target(case, seed):
    n = case["mesh"] // 4
    return 0.5 * torch.randn((n,) * 3, generator=_generator(seed + 5), device=DEV)


def prepare(case, seed):
    kind, P = case["kind"], _count(case)
    flags = {"run": 0, "power": 0, "learned": pm.PM_FLAG_LEARNED,
             "train": pm.PM_FLAG_LEARNED | pm.PM_FLAG_NO_SORT}.get(kind, pm.PM_FLAG_NO_SORT)
    s = dict(kind=kind, n=case["mesh"], ctx=pm.Ctx(pm.make_config(_config(case), flags=flags)), calls=_calls(case))
    if kind in ("run", "learned"):
        s["x0"], s["p0"], _ = _snapshot(case, seed)
        s["x"], s["p"] = torch.empty_like(s["x0"]), torch.empty_like(s["p0"])
        s["order"] = torch.arange(P, dtype=torch.int32, device=DEV)
        s["ids"] = torch.empty_like(s["order"])
        pm.pm_attach_ids(s["ctx"], s["ids"])
        s["theta"] = _theta(seed) if kind == "learned" else None
    elif kind == "train":
        s["x"], _, s["target"] = _snapshot(case, seed)
        s["theta0"], gen = _theta(seed), _generator(seed + 78)
        # Adam's moments a hundred steps into a training run
        s["m0"] = 1e-3 * torch.randn(s["theta0"].shape, generator=gen, device=DEV)
        s["v0"] = 1e-5 * torch.rand(s["theta0"].shape, generator=gen, device=DEV) + 1e-6
        s["a"] = case["a"]
        s.update({k: torch.empty_like(s["theta0"]) for k in ("theta", "m", "v", "g")})
    elif kind == "reconstruct":
        s["white"], s["target"] = _white(case, seed), _pool_target(case, seed)
    elif kind == "reverse":
        s["x0"], s["p0"], _ = _snapshot(case, seed)
        gen = _generator(seed + 79)
        s["xbar0"], s["pbar0"] = (torch.randn((3, P), generator=gen, device=DEV) for _ in range(2))
        s.update(x=torch.empty_like(s["x0"]), p=torch.empty_like(s["p0"]), xbar=torch.empty_like(s["x0"]),
                 pbar=torch.empty_like(s["x0"]))
    elif kind == "force":
        s["x"], _, _ = _snapshot(case, seed)
        s["acc"] = torch.empty_like(s["x"])
    elif kind == "ic":
        s["white"] = _white(case, seed)
        s["x"], s["p"] = s["ctx"].particles()
    else:
        s["x"], _, _ = _snapshot(case, seed)
        s["bins"], s["nseg"] = case["bins"], 1 + case["shell"]
    return s


# ---------------------------------------------------------------- a pass
def _moved(x, x0, n):
    """Periodic displacement from x0 to x."""
    return torch.remainder(x - x0 + 0.5 * n, float(n)) - 0.5 * n


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind in ("run", "learned"):
        x, p = s["x"], s["p"]
        x.copy_(s["x0"])
        p.copy_(s["p0"])
        s["ids"].copy_(s["order"])
        pm.pm_reset_order(ctx)
        for c in s["calls"]:
            if kind == "run":
                pm.pm_step(ctx, x, p, *c)
            else:
                pm.pm_learned_step(ctx, s["theta"], x, p, *c)
        back = s["ids"].long()
        xc, pc = torch.empty_like(x), torch.empty_like(p)
        xc[:, back] = x
        pc[:, back] = p
        return {"moved": _moved(xc, s["x0"], s["n"]), "p": pc}
    if kind == "train":
        for k in ("theta", "m", "v"):
            s[k].copy_(s[k + "0"])
        s["g"].zero_()
        loss = pm.pm_learned_loss(ctx, s["theta"], s["a"], s["x"], s["target"], s["g"])
        pm.pm_adam(s["theta"], s["m"], s["v"], s["g"], 1e-3, 0.9, 0.999, 1e-8, 100)
        # the forces carry float32, and so does the loss
        return {"loss": torch.tensor(loss, dtype=torch.float32), "g": s["g"], "theta": s["theta"], "m": s["m"],
                "v": s["v"]}
    if kind == "reconstruct":
        w = s["white"].clone().requires_grad_(True)
        delta = diff.final_density(ctx, w, s["calls"])
        pooled = torch.nn.functional.avg_pool3d(delta[None, None], 4)[0, 0]
        ((pooled - s["target"]) ** 2).sum().backward()
        return {"delta": delta.detach(), "g": w.grad}
    if kind == "reverse":
        for k in ("x", "p", "xbar", "pbar"):
            s[k].copy_(s[k + "0"])
        pm.pm_step(ctx, s["x"], s["p"], *s["calls"][0])
        pm.pm_step_vjp(ctx, s["x0"], *s["calls"][0], s["xbar"], s["pbar"])
        return {"moved": _moved(s["x"], s["x0"], s["n"]), "p": s["p"], "xbar": s["xbar"], "pbar": s["pbar"]}
    if kind == "force":
        pm.pm_force(ctx, s["x"], s["acc"])
        return {"acc": s["acc"]}
    if kind == "ic":
        pm.pm_ic(ctx, s["white"], s["x"], s["p"])
        return {"x": s["x"], "p": s["p"]}
    k, pt, modes = pm.pm_power(ctx, s["x"], 0, s["nseg"], nbins=s["bins"], compensate=True)
    _, pc, _ = pm.pm_power(ctx, s["x"], 0, 1, 1, s["nseg"], nbins=s["bins"])
    # the spectra carry the float32 of the meshes they come from
    return {"k": k, "modes": modes, "total": pt.astype(np.float32), "cross": pc.astype(np.float32)}


def work(case):
    kind, P, M, nc = case["kind"], float(_count(case)), float(case["mesh"]) ** 3, float(case["cdm"]) ** 3
    fft, cic = 2.5 * M * math.log2(M), 60.0 * P      # one real transform, one paint or three-component readout
    step = 4 * fft + 2 * cic + 12 * P
    net = 2.0 * 27 * (16 + 256 + 16) * M             # the three convolutions
    n_theta = 26818.0
    if kind == "run":
        return dict(bytes=case["calls"] * 48 * P, flops=case["calls"] * step)
    if kind == "learned":
        return dict(bytes=case["calls"] * 48 * P, flops=case["calls"] * (step + fft + net))
    if kind == "train":     # forward, and data and weight gradients
        return dict(bytes=24 * P + 40 * n_theta, flops=2 * step + 4 * fft + 3 * net)
    if kind == "reconstruct":
        return dict(bytes=8 * nc + 4 * M + case["calls"] * 96 * P, flops=3 * case["calls"] * step)
    if kind == "reverse":
        return dict(bytes=48 * P + 60 * P, flops=3 * step)
    if kind == "force":
        return dict(bytes=24 * P, flops=step)
    if kind == "ic":
        return dict(bytes=4 * nc + 24 * P, flops=7 * 2.5 * nc * math.log2(nc) + 30 * P)
    return dict(bytes=24 * P, flops=3 * fft + 2 * cic + 30 * M)


# ---------------------------------------------------------------- the same in 64 bits
class Background:
    """Expansion with Fermi-Dirac neutrinos and linear growth D, G = a^2 E dD/dlna."""

    def __init__(self, case):
        c, self.case = COSMO, case
        kT = 8.617333262e-5 * c["T_cmb"]
        rho = math.pi ** 2 / 15 * kT ** 4 / 1.973269804e-7 ** 3 * 1.602176634e-19 / 299792458.0 ** 2
        H = 1e5 / 3.0856775814913673e22
        self.og = rho / (3 * H * H / (8 * math.pi * 6.67430e-11)) / c["h"] ** 2
        self.m1 = case["m_nu"] / 3
        self.kT = kT * (4 / 11) ** (1 / 3) * (c["N_eff"] / 3) ** 0.25
        self.onu = case["m_nu"] / (93.14 * c["h"] ** 2)
        self.oc = c["omega_m"] - self.onu
        self.oL = 0.0
        self.oL = 1.0 - self.e2(np.array([1.0]))[0][0]
        h = 1e-3
        x0 = math.log(1 / 160)
        n = int(math.ceil((math.log(1.02) - x0) / h)) + 1
        self.x = x0 + h * np.arange(n)
        fine = x0 + 0.5 * h * np.arange(2 * n)
        e2, de2 = self.e2(np.exp(fine))
        fr, so = 2 + 0.5 * de2 / e2, 1.5 * c["omega_m"] * np.exp(-3 * fine) / e2
        y = np.array([1 / 160, 1 / 160])
        rhs = lambda j, v: np.array([v[1], so[j] * v[0] - fr[j] * v[1]])
        self.y, self.dy = np.empty((n, 2)), np.empty((n, 2))
        for i in range(n):
            k1 = rhs(2 * i, y)
            self.y[i], self.dy[i] = y, k1
            if i == n - 1:
                break
            k2 = rhs(2 * i + 1, y + 0.5 * h * k1)
            k3 = rhs(2 * i + 1, y + 0.5 * h * k2)
            y = y + h / 6 * (k1 + 2 * k2 + 2 * k3 + rhs(2 * i + 2, y + h * k3))

    def e2(self, a):
        x = np.linspace(0, 60, 3001)
        w = np.where(np.arange(3001) % 2, 4.0, 2.0)
        w[0] = w[-1] = 1.0
        w *= 0.02 / 3 * x * x / (1 + np.exp(x))
        pref = 15 / math.pi ** 4 * COSMO["N_eff"] / 3 * (4 / 11) ** (4 / 3) * self.og / a ** 4
        F, dF = np.empty_like(a), np.empty_like(a)
        for i in range(0, len(a), 512):
            y = (self.m1 * a[i:i + 512] / self.kT)[:, None]
            r = np.sqrt(x * x + y * y)
            F[i:i + 512] = r @ w
            dF[i:i + 512] = (y * y / np.maximum(r, 1e-300)) @ w
        return (self.og / a ** 4 + self.oc / a ** 3 + pref * 3 * F + self.oL,
                -4 * self.og / a ** 4 - 3 * self.oc / a ** 3 + pref * 3 * (dF - 4 * F))

    def DG(self, a):
        u = (math.log(a) - self.x[0]) / 1e-3
        i = min(int(u), len(self.x) - 2)
        t = u - i
        b = np.array([2 * t ** 3 - 3 * t ** 2 + 1, 3 * t ** 2 - 2 * t ** 3])
        d = 1e-3 * np.array([t ** 3 - 2 * t ** 2 + t, t ** 3 - t ** 2])
        D, Dp = b @ self.y[i:i + 2] + d @ self.dy[i:i + 2]
        return D, a * a * math.sqrt(self.e2(np.array([a]))[0][0]) * Dp

    def factors(self, call):
        af, k0, k1, d1 = call
        D, G1 = self.DG(af)[0], self.DG(k1)[1]
        return (G1 - self.DG(k0)[1]) / (1.5 * COSMO["omega_m"] * D), (self.DG(d1)[0] - D) / G1

    def shells(self):
        """(speeds, mass fractions) of the neutrino shells: equal area under q f(q)."""
        q = np.linspace(0, 30, 1_200_001)
        f, h = 1 / (np.exp(q) + 1), q[1]
        cum = lambda g: np.concatenate([[0], np.cumsum((g[:-1] + g[1:]) * (h / 2) - np.diff(np.gradient(g, h)) * h * h / 12)])
        c1, c2, c4 = cum(q * f), cum(q ** 2 * f), cum(q ** 4 * f)
        edge = np.interp(np.linspace(0, 1, self.case["shell"] + 1) * c1[-1], c1, q)
        m2, m4 = (np.diff(np.interp(edge, q, c)) for c in (c2, c4))
        return np.sqrt(m4 / m2), m2 / m2.sum()

    def masses(self):
        """Mass per particle, float64 [P] (mean of one per cell)."""
        c, M = self.case, float(self.case["mesh"]) ** 3
        nd = 2 * c["fib"] + 1
        m = [torch.full((c["cdm"] ** 3,), self.oc / COSMO["omega_m"] * M / c["cdm"] ** 3, dtype=torch.float64, device=DEV)]
        for f in self.shells()[1]:
            m.append(torch.full((c["sites"] ** 3 * nd,), self.onu / COSMO["omega_m"] * M / c["sites"] ** 3 * f / nd,
                                dtype=torch.float64, device=DEV))
        return torch.cat(m)


def _modes(n):
    """Wave vectors in grid units, each zero on its own Nyquist frequency (for
    gradients), and k^2 with the true ones (1 at k = 0)."""
    f = torch.fft.fftfreq(n, dtype=torch.float64, device=DEV) * 2 * math.pi
    r = torch.fft.rfftfreq(n, dtype=torch.float64, device=DEV) * 2 * math.pi
    kk = f[:, None, None] ** 2 + f[None, :, None] ** 2 + r[None, None, :] ** 2
    kk[0, 0, 0] = 1.0
    f, r = f.clone(), r.clone()
    f[n // 2] = 0
    r[n // 2] = 0
    return (f[:, None, None], f[None, :, None], r[None, None, :]), kk


def _corners(x, n):
    i = torch.floor(x.detach())
    f = x - i
    i = i.long()
    for a in (0, 1):
        for b in (0, 1):
            for c in (0, 1):
                idx = (((i[0] + a) % n) * n + (i[1] + b) % n) * n + (i[2] + c) % n
                yield idx, ((f[0] if a else 1 - f[0]) * (f[1] if b else 1 - f[1])) * (f[2] if c else 1 - f[2])


def _delta(x, m, n):
    rho = torch.zeros(n ** 3, dtype=torch.float64, device=DEV)
    for idx, w in _corners(x, n):
        rho = rho.index_add(0, idx, m * w) if x.requires_grad else rho.index_add_(0, idx, m * w)
    return (rho - 1).reshape(n, n, n)


def _readout(fields, x, n):
    acc = [0.0, 0.0, 0.0]
    for idx, w in _corners(x, n):
        for d in range(3):
            acc[d] = acc[d] + w * fields[d].reshape(-1)[idx]
    return torch.stack(acc)


def _gradient(pk, n, k):
    """-grad of the potential with spectrum pk."""
    return [torch.fft.irfftn(-1j * k[d] * pk, s=(n, n, n)) for d in range(3)]


def _force(x, m, n):
    k, kk = _modes(n)
    pk = torch.fft.rfftn(_delta(x, m, n)) * (-1.5 * COSMO["omega_m"] / kk)
    return _readout(_gradient(pk, n, k), x, n)


class Conv(torch.autograd.Function):
    """Periodic 3^3 convolution [ci, n, n, n] -> [co, n, n, n], weights [co, ci, 27]."""

    @staticmethod
    def shift(a, t, sign):
        return torch.roll(a, [-sign * (t // 9 - 1), -sign * (t // 3 % 3 - 1), -sign * (t % 3 - 1)], (1, 2, 3))

    @staticmethod
    def forward(fctx, a, w):
        fctx.save_for_backward(a, w)
        n = a.shape[1]
        out = torch.zeros((w.shape[0], n ** 3), dtype=torch.float64, device=DEV)
        for t in range(27):
            out.addmm_(w[:, :, t], Conv.shift(a, t, 1).reshape(a.shape[0], -1))
        return out.reshape(-1, n, n, n)

    @staticmethod
    def backward(fctx, g):
        a, w = fctx.saved_tensors
        gm = g.reshape(g.shape[0], -1)
        dw = torch.stack([gm @ Conv.shift(a, t, 1).reshape(a.shape[0], -1).T for t in range(27)], -1)
        da = None
        if fctx.needs_input_grad[0]:
            da = torch.zeros((a.shape[0], gm.shape[1]), dtype=torch.float64, device=DEV)
            for t in range(27):
                da.addmm_(w[:, :, t].T.contiguous(), Conv.shift(g, t, -1).reshape(g.shape[0], -1))
            da = da.reshape(a.shape)
        return da, dw


def _parts(theta):
    out, o = [], 0
    for shape in ((96, 2), (96,), (96, 96), (96,), (96, 96), (96,), (96,), (1,), (16, 1, 27), (16,), (16, 16, 27), (16,),
                  (1, 16, 27), (1,)):
        size = math.prod(shape)
        out.append(theta[o:o + size].reshape(shape))
        o += size
    return out


def _learned_force(theta, a, x, m, n):
    w0, b0, w1, b1, w2, b2, w3, b3, c1, d1, c2, d2, c3, d3 = _parts(theta)
    silu = torch.nn.functional.silu
    kt = torch.arange(256, dtype=torch.float64, device=DEV) * math.sqrt(3) / 255
    h = silu(torch.stack([kt, torch.full_like(kt, a)], 1) @ w0.T + b0)
    table = 1 + silu(silu(h @ w1.T + b1) @ w2.T + b2) @ w3 + b3
    delta = _delta(x, m, n)
    k, kk = _modes(n)
    t = torch.sqrt(kk) / math.pi * 255 / math.sqrt(3)
    i = t.long().clamp(max=254)
    g = table[i] * (1 - (t - i)) + table[i + 1] * (t - i)
    filtered = torch.fft.rfftn(delta) * (-1.5 * COSMO["omega_m"] / kk) * g
    keep = torch.ones_like(kk)
    keep[0, 0, 0] = 0
    filtered = filtered * keep
    y = silu(Conv.apply(delta[None], c1) + d1[:, None, None, None])
    y = silu(Conv.apply(y, c2) + d2[:, None, None, None])
    cnn = (Conv.apply(y, c3) + d3[:, None, None, None])[0]
    return _readout(_gradient(filtered + torch.fft.rfftn(cnn), n, k), x, n)


def _ic(case, bg, white):
    """Zel'dovich initial conditions (x before the wrap, p), float64 [3, P]."""
    nc, n, box, a0 = case["cdm"], case["mesh"], case["box"], _config(case)["a0"]
    (D0, G0), D1 = bg.DG(a0), bg.DG(1.0)[0]
    omh = COSMO["omega_m"] * COSMO["h"]

    def transfer(q, lib):
        poly = 1 + 3.89 * q + (16.1 * q) ** 2 + (5.46 * q) ** 3 + (6.71 * q) ** 4
        return lib.log(1 + 2.34 * q) / (2.34 * q) * poly ** -0.25

    lk = np.linspace(math.log(1e-6), math.log(1e3), 400001)
    kq, simpson = np.exp(lk), np.where(np.arange(400001) % 2, 4.0, 2.0)
    simpson[0] = simpson[-1] = 1.0
    r = 8 * kq
    win = np.where(r < 1e-3, 1 - r * r / 10, 3 * (np.sin(r) - r * np.cos(r)) / r ** 3)
    s2 = np.sum(simpson * kq ** (3 + COSMO["n_s"]) * transfer(kq / omh, np) ** 2 * win ** 2) * (lk[1] - lk[0]) / 3
    A = COSMO["sigma8"] ** 2 / (s2 / (2 * math.pi ** 2))
    k, kk = _modes(nc)
    s = nc / box
    kp = torch.sqrt(kk) * s
    amp = torch.sqrt(A * (D0 / D1) ** 2 / (box / nc) ** 3 * kp ** COSMO["n_s"]) * transfer(kp / omh, torch)
    edge = torch.zeros(nc, dtype=torch.bool, device=DEV)
    edge[nc // 2] = True
    drop = edge[:, None, None] | edge[None, :, None] | edge[None, None, :nc // 2 + 1]
    drop[0, 0, 0] = True
    spec = torch.where(drop, 0.0, torch.fft.rfftn(white) * amp) * (n / box)
    field = lambda sp: torch.stack([torch.fft.irfftn(1j * k[d] / (kk * s) * sp, s=(nc,) * 3) for d in range(3)])
    sc = field(spec).reshape(3, -1)
    i = torch.arange(nc, dtype=torch.float64, device=DEV) * (n / nc)
    lat = torch.stack(torch.meshgrid(i, i, i, indexing="ij")).reshape(3, -1)
    x, p = [lat + sc], [G0 / D0 * sc]
    ns, R, nd = case["sites"], nc // case["sites"], 2 * case["fib"] + 1
    kfs = 0.82 * math.sqrt(bg.oL + COSMO["omega_m"] / a0 ** 3) * a0 ** 2 * bg.m1
    sn = field(spec / (1 + (kp / kfs) ** 2) * torch.exp(0.5j * (k[0] + k[1] + k[2])))
    at = torch.arange(ns, device=DEV) * R + R // 2
    sn = sn[:, at[:, None, None], at[None, :, None], at[None, None, :]].reshape(3, -1, 1)
    c = (at + 0.5) * (n / nc)
    centre = torch.stack(torch.meshgrid(c, c, c, indexing="ij")).reshape(3, -1, 1)
    j = torch.arange(ns, device=DEV)
    flip = 1.0 - 2.0 * ((j[:, None, None] + j[None, :, None] + j[None, None, :]) % 2).double().reshape(-1, 1)
    t = torch.arange(-case["fib"], case["fib"] + 1, dtype=torch.float64, device=DEV)
    lat_, lon = torch.asin(2 * t / nd), 4 * math.pi / (1 + math.sqrt(5)) * t
    v = torch.stack([torch.cos(lat_) * torch.cos(lon), torch.cos(lat_) * torch.sin(lon), torch.sin(lat_)])
    speed = bg.shells()[0]
    for q in speed:
        d = flip * v[:, None, :]
        x.append((centre + 0.4 * n / ns * q / speed[-1] * d + sn).reshape(3, -1))
        p.append((q * bg.kT / bg.m1 * 2997.92458 * n / box * d + G0 / D0 * sn).reshape(3, -1))
    return torch.cat(x, 1), torch.cat(p, 1)


def _reconstruct_exact(case, bg, m, white, target):
    n = case["mesh"]
    w = white.double().requires_grad_(True)
    x, p = _ic(case, bg, w)
    for c in _calls(case):
        kick, drift = bg.factors(c)
        x = x - torch.floor(x.detach() / n) * n
        p = p + kick * _force(x, m, n)
        x = x + drift * p
    delta = _delta(x - torch.floor(x.detach() / n) * n, m, n)
    pooled = torch.nn.functional.avg_pool3d(delta[None, None], 4)[0, 0]
    ((pooled - target.double()) ** 2).sum().backward()
    return {"delta": delta.detach(), "g": w.grad}


def exact(case, seed):
    kind, n = case["kind"], case["mesh"]
    bg = Background(case)
    m = bg.masses()
    if kind in ("run", "learned"):
        x0, p, _ = _snapshot(case, seed)
        x, p = x0.double(), p.double()
        theta = _theta(seed).double() if kind == "learned" else None
        with torch.no_grad():
            for c in _calls(case):
                kick, drift = bg.factors(c)
                p = p + kick * (_force(x, m, n) if theta is None else _learned_force(theta, c[0], x, m, n))
                x = torch.remainder(x + drift * p, n)
        return {"moved": _moved(x, x0.double(), n), "p": p}
    if kind == "train":
        x, _, target = _snapshot(case, seed)
        theta, gen = _theta(seed).double().requires_grad_(True), _generator(seed + 78)
        m0 = 1e-3 * torch.randn(theta.shape, generator=gen, device=DEV).double()
        v0 = (1e-5 * torch.rand(theta.shape, generator=gen, device=DEV) + 1e-6).double()
        acc = _learned_force(theta, case["a"], x.double(), m, n)
        loss = ((acc - target) ** 2).sum() / (target.double() ** 2).sum()
        loss.backward()
        g = theta.grad
        m1, v1 = 0.9 * m0 + 0.1 * g, 0.999 * v0 + 0.001 * g * g
        th = theta.detach() - 1e-3 * (m1 / (1 - 0.9 ** 100)) / (torch.sqrt(v1 / (1 - 0.999 ** 100)) + 1e-8)
        return {"loss": loss.detach(), "g": g, "theta": th, "m": m1, "v": v1}
    if kind == "reconstruct":
        return _reconstruct_exact(case, bg, m, _white(case, seed), _pool_target(case, seed))
    if kind == "reverse":
        x0, p0, _ = _snapshot(case, seed)
        gen = _generator(seed + 79)
        xbar, pbar = (torch.randn(x0.shape, generator=gen, device=DEV).double() for _ in range(2))
        x, p = x0.double().requires_grad_(True), p0.double().requires_grad_(True)
        kick, drift = bg.factors(_calls(case)[0])
        p1 = p + kick * _force(x, m, n)
        x1 = x + drift * p1
        torch.autograd.backward([x1, p1], [xbar, pbar])
        return {"moved": _moved(x1.detach(), x0.double(), n), "p": p1.detach(), "xbar": x.grad, "pbar": p.grad}
    if kind == "force":
        with torch.no_grad():
            return {"acc": _force(_snapshot(case, seed)[0].double(), m, n)}
    if kind == "ic":
        x, p = _ic(case, bg, _white(case, seed).double())
        return {"x": _wrap(torch.remainder(x, n).float(), n).double(), "p": p}
    x = _snapshot(case, seed)[0].double()
    c, full = case["cdm"] ** 3, n ** 3
    f = torch.fft.fftfreq(n, 1 / n, dtype=torch.float64, device=DEV)
    f = [f[:, None, None], f[None, :, None], f[None, None, :n // 2 + 1].abs()]
    nn = f[0] ** 2 + f[1] ** 2 + f[2] ** 2
    bins = torch.floor(torch.sqrt(nn)).long()
    weight = torch.where((f[2] == 0) | (f[2] == n // 2), 1.0, 2.0).double().expand(nn.shape).clone()
    weight[0, 0, 0] = 0

    def binned(v):
        return torch.bincount(bins.reshape(-1), (weight * v).reshape(-1), minlength=case["bins"])[:case["bins"]].cpu().numpy()

    def spectrum(lo, hi):
        return torch.fft.rfftn(_delta(x[:, lo:hi], m[lo:hi] * (full / m[lo:hi].sum()), n))

    window = 1.0
    for d in range(3):
        window = window * torch.sinc(f[d] / n) ** 4
    A = spectrum(0, x.shape[1])
    modes = binned(torch.ones_like(nn))
    total = binned((A.real ** 2 + A.imag ** 2) / window)
    A, B = spectrum(0, c), spectrum(c, x.shape[1])
    cross = binned(A.real * B.real + A.imag * B.imag)
    norm = case["box"] ** 3 / full ** 2 / np.maximum(modes, 1)
    return {"k": binned(torch.sqrt(nn)) * 2 * math.pi / case["box"] / np.maximum(modes, 1), "modes": modes,
            "total": total * norm, "cross": cross * norm}
