"""Workloads the solver is measured on: what a program on top of the library has it do,
through its public entry points (Solver, Batch, evolve_real).

A pass of a "run" case is one output interval of a simulation: load a state that is on the
GPU, take the interval's imaginary- or real-time steps, read the observables and the wave
function.  "gradient" is one forward and backward pass of an optimisation over initial state,
trap and couplings; "ensemble" is one output interval of many independent planar systems.
The references below are plain torch in 64 bits: Crank-Nicolson factors as dense matrices
from the eigenvectors of the second difference, the dipolar term by torch.fft.
"""
from __future__ import annotations

import math
import random

import torch
import torch.utils.checkpoint

DEV = "cuda:0"
# even 2^a 3^b 5^c lengths that every entry point takes, the adjoint and the ensemble too
ADJOINT_SIZES = (32, 48, 64, 80, 96, 120, 128, 160, 192)
ENSEMBLE_SIZES = (96, 128, 192, 256, 384, 512)


# ------------------------------------------------------------------------------- cases
def _run(name, geom, n, prec, imag, steps, trap="harmonic"):
    c = dict(kind="run", geom=geom, nx=n[0], ny=n[1], nz=n[2], prec=prec, imag=imag, steps=steps, trap=trap)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a small planar system, a few relaxation steps between two
        # readings (an interactive or feedback loop); launches and latency count
        _run("2dxy_96x80_fp64_imag", "2dxy", (96, 80, 1), "fp64", True, 10),
        # the repository's planar real-time workload: 256 x 256 in a perturbed trap
        _run("2dxy_256_fp32_real", "2dxy", (256, 256, 1), "fp32", False, 200, "perturbed"),
        # planar ground state on a grid that is no power of two
        _run("2dxz_540x600_fp64_imag", "2dxz", (540, 1, 600), "fp64", True, 60),
        # a wide, finely resolved planar cloud
        _run("2dxy_2000x1500_fp32_real", "2dxy", (2000, 1500, 1), "fp32", False, 40),
        # the small 3D ground-state search
        _run("3d_64_fp64_imag", "3d", (64, 64, 64), "fp64", True, 100),
        # the medium 3D quench in mixed precision
        _run("3d_128x96x80_fp32_real", "3d", (128, 96, 80), "fp32", False, 100),
        # odd, ragged lengths (the grid is never padded or enlarged); 101 is a prime
        _run("3d_101x75x63_fp32_imag", "3d", (101, 75, 63), "fp32", True, 40),
        # a round length that is not a power of two, full precision
        _run("3d_200_fp64_real", "3d", (200, 200, 200), "fp64", False, 10),
        # the headline grid
        _run("3d_256_fp64_real", "3d", (256, 256, 256), "fp64", False, 16),
        # the largest: a production-size relaxation
        _run("3d_400_fp32_imag", "3d", (400, 400, 400), "fp32", True, 8),
        # gradients of a control problem: 3D, checkpoints every 10 steps
        dict(name="3d_128_fp64_gradient", kind="gradient", geom="3d", nx=128, ny=128, nz=128, prec="fp64",
             steps=20, every=10),
        # many small planar systems of uneven size, relaxed together
        dict(name="ensemble_192_fp32_imag", kind="ensemble", count=192, prec="fp32", imag=True, steps=160, mix=1606),
    ]


def _length(rng, lo, hi):
    """An axis length as people choose it, over the logarithm of the range: a product of 2, 3
    and 5, a round decimal number, or any number at all."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    how = rng.random()
    if how < 0.45:
        fives = [2 ** a * 3 ** b * 5 ** c for a in range(1, 13) for b in range(4) for c in range(4)]
        n = min((m for m in fives if lo <= m <= hi), key=lambda m: abs(math.log(m / n)))
    elif how < 0.75:
        n = max(lo, min(hi, 10 * round(n / 10)))
    return n


def draw(rng):
    what = rng.random()
    prec = rng.choice(("fp64", "fp32"))
    if what < 0.08:
        n = [rng.choice(ADJOINT_SIZES) for _ in range(3)]
        steps = rng.randint(8, 20)
        return dict(kind="gradient", geom="3d", nx=min(n[0], 128), ny=n[1], nz=min(n[2], 128), prec=prec,
                    steps=steps, every=rng.randint(4, 10))
    if what < 0.16:
        return dict(kind="ensemble", count=rng.randint(12, 96), prec=prec, imag=rng.random() < 0.5,
                    steps=rng.randint(16, 40), mix=rng.randrange(1 << 20))
    imag = rng.random() < 0.5
    trap = rng.choice(("harmonic", "perturbed"))
    if what < 0.5:
        geom = rng.choice(("2dxy", "2dxz"))
        a, b = _length(rng, 64, 2000), _length(rng, 64, 2000)
        n = (a, b, 1) if geom == "2dxy" else (a, 1, b)
    else:
        geom = "3d"
        while True:
            n = tuple(_length(rng, 32, 400) for _ in range(3))
            if n[0] * n[1] * n[2] <= 30_000_000:
                break
    pts = n[0] * n[1] * n[2]
    most = max(6, min(200, int(1.5e8 / pts)))
    return _run(None, geom, n, prec, imag, rng.randint(max(5, most // 2), most), trap)


# ------------------------------------------------------------------------------ inputs
def _params(case):
    """Physical parameters of a run or gradient case."""
    p = {k: case[k] for k in ("geom", "nx", "ny", "nz")}
    if p["geom"] == "3d":
        box = 16.0
        p.update(dx=box / p["nx"], dy=box / p["ny"], dz=box / p["nz"], dt=0.001, gamma=1.0, nu=1.0,
                 lam=2.0, g=20.0, gdd=6.0, R=8.0)
    else:
        box = 25.6
        p.update(dx=box / p["nx"], dy=box / max(p["ny"], p["nz"]), dz=box / max(p["ny"], p["nz"]),
                 dt=0.0005, gamma=1.0, R=0.0, g=30.0, gdd=10.0)
        p.update(dict(nu=1.5, lam=4.0) if p["geom"] == "2dxy" else dict(nu=4.0, lam=1.5))
    return p


def _axes(p):
    """(length, spacing, trap frequency) in array order, slowest first."""
    x = (p["nx"], p["dx"], p["gamma"])
    y = (p["ny"], p["dy"], p["nu"])
    z = (p["nz"], p["dz"], p["lam"])
    return {"3d": (z, y, x), "2dxy": (y, x), "2dxz": (z, x)}[p["geom"]]


def _coords(p):
    ax = _axes(p)
    return [((torch.arange(n, dtype=torch.float64, device=DEV) - n // 2) * h).reshape(
        [-1 if i == k else 1 for i in range(len(ax))]) for k, (n, h, _) in enumerate(ax)]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _start(p, gen):
    """A normalised cloud of the trap's shape with 1 % amplitude and 0.5 % phase noise, zero
    on the boundary."""
    x, ax = _coords(p), _axes(p)
    psi = torch.ones([n for n, _, _ in ax], dtype=torch.float64, device=DEV)
    for c, (_, _, w) in zip(x, ax):
        psi = psi * torch.exp(-0.5 * w * c * c)
    u = 2 * torch.rand(2, *psi.shape, dtype=torch.float64, device=DEV, generator=gen) - 1
    psi = torch.polar(psi * (1 + 0.01 * u[0]), 2 * math.pi * 0.005 * u[1])
    psi = _inner(psi)
    return psi / torch.sqrt((psi.real ** 2 + psi.imag ** 2).sum() * _cell(p))


def _inner(a):
    for k in range(a.ndim):
        a.select(k, 0).zero_()
        a.select(k, a.shape[k] - 1).zero_()
    return a


def _cell(p):
    return math.prod(h for _, h, _ in _axes(p))


def _trap(p, case, gen):
    """The harmonic trap, or that trap with a smooth random perturbation of rms 0.1."""
    v = sum(0.5 * (w * c) ** 2 for c, (_, _, w) in zip(_coords(p), _axes(p)))
    if case.get("trap") != "perturbed":
        return v
    f = torch.randn(v.shape, dtype=torch.float64, device=DEV, generator=gen)
    k2 = 0
    for i, (n, h, _) in enumerate(_axes(p)):
        k = 2 * math.pi * torch.fft.fftfreq(n, d=h, dtype=torch.float64, device=DEV)
        k2 = k2 + (k * k).reshape([-1 if i == j else 1 for j in range(v.ndim)])
    f = torch.fft.ifftn(torch.fft.fftn(f) * torch.exp(-0.5 * k2)).real
    return v + 0.1 * f / torch.sqrt((f * f).mean())


def _target(p, gen):
    """A displaced cloud: the state a control problem steers to."""
    off = (torch.rand(len(_axes(p)), dtype=torch.float64, device=DEV, generator=gen) - 0.5).tolist()
    t = 1.0
    for c, o, (_, _, w) in zip(_coords(p), off, _axes(p)):
        t = t * torch.exp(-0.5 * w * (c - o) ** 2)
    t = _inner(t.to(torch.complex128))
    return t / torch.sqrt((t.real ** 2).sum() * _cell(p))


def _ensemble(case):
    r, out = random.Random(case["mix"]), []
    for i in range(case["count"]):
        n0, n1 = r.choice(ENSEMBLE_SIZES), r.choice(ENSEMBLE_SIZES)
        a, h = r.uniform(0.5, 4.0), r.uniform(0.05, 0.2)
        p = dict(dx=h, dy=h, dz=h, dt=0.001, gamma=1.0, g=r.uniform(0, 50), gdd=r.uniform(0, 30), R=0.0)
        if i % 2:
            p.update(geom="2dxz", nx=n0, ny=1, nz=n1, nu=4.0, lam=a)
        else:
            p.update(geom="2dxy", nx=n0, ny=n1, nz=1, nu=a, lam=4.0)
        out.append(p)
    return out


def _types(case):
    return (torch.complex128, torch.float64) if case["prec"] == "fp64" else (torch.complex64, torch.float32)


def prepare(case, seed):
    from paper_1601_04640_amd.binding import Batch, Solver
    gen, (ct, rt) = _gen(seed), _types(case)
    if case["kind"] == "ensemble":
        ps = _ensemble(case)
        batch = Batch(ps, prec=case["prec"])
        return dict(case=case, batch=batch, psi0=[_start(p, gen).to(ct) for p in ps])
    p = _params(case)
    solver = Solver(p, prec=case["prec"])
    psi0 = _start(p, gen)
    v = _trap(p, case, gen)
    if case["kind"] == "gradient":
        leaf = lambda x: torch.tensor(x, dtype=torch.float64, device=DEV, requires_grad=True)  # noqa: E731
        return dict(case=case, p=p, solver=solver, psi0=psi0.to(ct).requires_grad_(True),
                    v=v.requires_grad_(True), g=leaf(p["g"]), gdd=leaf(p["gdd"]), target=_target(p, gen).to(ct))
    if case["trap"] == "perturbed":
        solver.set_potential(v.to(rt))
    return dict(case=case, solver=solver, psi0=psi0.to(ct))


# -------------------------------------------------------------------------------- run
def _record(o):
    return [o["norm"], o["mu"], o["energy"], o["e_kin"], o["e_pot"], o["e_int"], o["e_dd"], *o["rms"]]


def run(state):
    case = state["case"]
    rt = _types(case)[1]
    if case["kind"] == "ensemble":
        from paper_1601_04640_amd.binding import gp_get_psi
        b = state["batch"]
        for i, psi in enumerate(state["psi0"]):
            b.set_psi(i, psi)
        (b.step_imag if case["imag"] else b.step_real)(case["steps"])
        obs = torch.tensor([_record(o) for o in b.energy()], dtype=rt)
        out = torch.empty(b.points(), dtype=state["psi0"][0].dtype, device=DEV)
        at = 0
        for i, psi in enumerate(state["psi0"]):
            gp_get_psi(b.ctxs[i], out[at:].data_ptr(), 1)
            at += psi.numel()
        return dict(observables=obs, psi=out)
    s = state["solver"]
    if case["kind"] == "gradient":
        from paper_1601_04640_amd.adjoint import evolve_real, overlap_loss
        xs = [state[k] for k in ("psi0", "v", "g", "gdd")]
        psi = evolve_real(s, *xs, case["steps"], case["every"])
        loss = overlap_loss(psi, state["target"], _cell(state["p"]))
        grads = torch.autograd.grad(loss, xs)
        # the gradients of a single-precision evolution are single precision, however wide
        # the accumulators they are handed back in
        return dict(loss=loss.detach(), psi0=grads[0],
                    v=grads[1].to(rt), couplings=torch.stack(grads[2:]).to(rt))
    s.set_psi(state["psi0"])
    (s.step_imag if case["imag"] else s.step_real)(case["steps"])
    obs = torch.tensor(_record(s.energy()), dtype=rt)
    return dict(observables=obs, psi=s.get_psi_device())


# ------------------------------------------------------------------------------- work
def _step_work(shape, prec, imag):
    """A step reads psi and the trap and writes psi; two real transforms, the phase, and a
    tridiagonal solve per axis (a multiply and an add of a complex value forward and back,
    real factors in imaginary time)."""
    n, r = math.prod(shape), 8 if prec == "fp64" else 4
    fft = 2 * 2.5 * n * math.log2(n)
    return n * 5 * r, fft + n * (30 + len(shape) * (14 if imag else 26))


def work(case):
    if case["kind"] == "ensemble":
        one = [_step_work([a[0] for a in _axes(p)], case["prec"], case["imag"]) for p in _ensemble(case)]
        steps = case["steps"]
    else:
        one = [_step_work([a[0] for a in _axes(_params(case))], case["prec"], case.get("imag", False))]
        # backward recomputes the states between the checkpoints and takes a costate through
        # each step (it has two convolutions)
        steps = case["steps"] * (4 if case["kind"] == "gradient" else 1)
    return dict(bytes=float(steps * sum(b for b, _ in one)), flops=float(steps * sum(f for _, f in one)))


# ------------------------------------------------------------------------------ exact
def _kernel(p):
    """U(k) on the half spectrum (last axis x)."""
    ax = _axes(p)
    ks = []
    for i, (n, h, _) in enumerate(ax):
        f = torch.fft.rfftfreq if i == len(ax) - 1 else torch.fft.fftfreq
        ks.append((2 * math.pi * f(n, d=h, dtype=torch.float64, device=DEV)).reshape(
            [-1 if i == j else 1 for j in range(len(ax))]))
    q2 = sum(k * k for k in ks)
    safe = torch.where(q2 > 0, q2, 1.0)
    if p["geom"] == "3d":
        u = 3 * ks[0] ** 2 / safe - 1
        s = torch.sqrt(safe) * p["R"]
        big = 1 + 3 * torch.cos(s) / s ** 2 - 3 * torch.sin(s) / s ** 3
        t = torch.minimum(s, torch.ones_like(s)) ** 2
        small = torch.zeros_like(s)
        for k in range(2, 14):  # sum (-1)^k 6k s^(2k-2) / (2k+1)!
            small = small + t ** (k - 1) * ((-1) ** k * 6 * k / math.factorial(2 * k + 1))
        return torch.where(q2 > 0, u * torch.where(s < 1, small, big), 0.0)
    d = 1 / math.sqrt(p["lam"] if p["geom"] == "2dxy" else p["nu"])
    xi = torch.sqrt(q2) * d / math.sqrt(2)
    ex = 3 * math.sqrt(math.pi) * xi * torch.special.erfcx(xi)
    u = 2 - ex if p["geom"] == "2dxy" else -1 + torch.where(q2 > 0, ks[0] ** 2 / safe, 0.0) * ex
    return u / (math.sqrt(2 * math.pi) * d)


def _contact(p):
    if p["geom"] == "3d":
        return 1.0
    return math.sqrt(p["lam"] if p["geom"] == "2dxy" else p["nu"]) / math.sqrt(2 * math.pi)


def _factor(n, h, dt, imag):
    """(1 + A T)^-1 (1 - A T) on the inner points, T = tridiag(-1, 2, -1), A = eps dt/(4 h^2)."""
    k = torch.arange(1, n - 1, dtype=torch.float64, device=DEV)
    s = math.sqrt(2 / (n - 1)) * torch.sin(math.pi / (n - 1) * torch.outer(k, k).remainder(2 * (n - 1)))
    a = dt / (4 * h * h) * (1.0 if imag else 1j) * (2 - 2 * torch.cos(math.pi * k / (n - 1)))
    m = torch.zeros(n, n, dtype=torch.complex128, device=DEV)
    m[1:-1, 1:-1] = (s * ((1 - a) / (1 + a))).to(m.dtype) @ s.to(m.dtype)
    return m


class _Exact:
    def __init__(self, p, imag):
        self.p, self.imag, self.cell, self.ker = p, imag, _cell(p), _kernel(p)
        self.m = [_factor(n, h, p["dt"], imag) for n, h, _ in _axes(p)]

    def phi(self, n):
        return torch.fft.irfftn(torch.fft.rfftn(n) * self.ker, s=n.shape)

    def step(self, psi, v, g, gdd):
        n = psi.real ** 2 + psi.imag ** 2
        th = self.p["dt"] * (v + g * _contact(self.p) * n + gdd * self.phi(n))
        psi = psi * (torch.exp(-th) if self.imag else torch.polar(torch.ones_like(th), -th))
        psi = psi @ self.m[-1].T
        if psi.ndim == 3:
            psi = torch.matmul(self.m[1], psi)
        psi = (self.m[0] @ psi.reshape(psi.shape[0], -1)).reshape(psi.shape)
        if self.imag:
            psi = psi / torch.sqrt((psi.real ** 2 + psi.imag ** 2).sum() * self.cell)
        return psi

    def observables(self, psi, v):
        p, dv = self.p, self.cell
        n = psi.real ** 2 + psi.imag ** 2
        kin = 0
        for k, (_, h, _) in enumerate(_axes(p)):
            d = torch.diff(psi, dim=k)
            kin = kin + 0.5 * (d.real ** 2 + d.imag ** 2).sum() / (h * h) * dv
        norm, pot = n.sum() * dv, (v * n).sum() * dv
        con = 0.5 * p["g"] * _contact(p) * (n * n).sum() * dv
        dd = 0.5 * p["gdd"] * (self.phi(n) * n).sum() * dv
        rms = [torch.sqrt((c * c * n).sum() * dv / norm) for c in _coords(p)][::-1]
        zero = torch.zeros_like(norm)
        rms = {"3d": rms, "2dxy": [*rms, zero], "2dxz": [rms[0], zero, rms[-1]]}[p["geom"]]
        return torch.stack([norm, kin + pot + 2 * con + 2 * dd, kin + pot + con + dd, kin, pot, con, dd, *rms])


def exact(case, seed):
    gen, (ct, rt) = _gen(seed), _types(case)
    if case["kind"] == "ensemble":
        obs, out = [], []
        for p in _ensemble(case):
            psi, e, v = _start(p, gen).to(ct).to(torch.complex128), _Exact(p, case["imag"]), _trap(p, {}, None)
            for _ in range(case["steps"]):
                psi = e.step(psi, v, p["g"], p["gdd"])
            obs.append(e.observables(psi, v))
            out.append(psi.reshape(-1))
        return dict(observables=torch.stack(obs).cpu(), psi=torch.cat(out))
    p = _params(case)
    psi = _start(p, gen).to(ct).to(torch.complex128)
    v = _trap(p, case, gen)
    e = _Exact(p, case.get("imag", False))
    if case["kind"] == "gradient":
        xs = [psi.requires_grad_(True), v.requires_grad_(True)] + [
            torch.tensor(p[k], dtype=torch.float64, device=DEV, requires_grad=True) for k in ("g", "gdd")]
        target = _target(p, gen).to(ct).to(torch.complex128)
        for _ in range(case["steps"]):
            psi = torch.utils.checkpoint.checkpoint(e.step, psi, *xs[1:], use_reentrant=False)
        c = (torch.conj(target) * psi).sum() * e.cell
        loss = 1 - (c.real ** 2 + c.imag ** 2)
        grads = torch.autograd.grad(loss, xs)
        return dict(loss=loss.detach(), psi0=grads[0], v=grads[1], couplings=torch.stack(grads[2:]))
    if case["trap"] == "perturbed":
        v = v.to(rt).to(torch.float64)
    for _ in range(case["steps"]):
        psi = e.step(psi, v, p["g"], p["gdd"])
    return dict(observables=e.observables(psi, v).cpu(), psi=psi)
