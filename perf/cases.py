"""Performance cases of the multigrid library: what simulation codes ask of it.

A particle-mesh code solves the seven-point Poisson problem once per time
step, starting from the previous potential; a moving-mesh code rebuilds the
geometry, solves the 19-point flux-form problem and reads the force; an
inference code differentiates that chain.  Every case is one such call, or
one such step, through the public Python entry points.

Grids are n^3 with n a power of two (nothing else is accepted); what varies
beside n is the number of levels, the smoother and its degree, the precision,
the spacing, the tolerance or the number of cycles, and the spectra of the
inputs.  All inputs are Gaussian random fields made on the GPU from the seed.
Warm starts are exact: the previous potential phi_prev is drawn, its source
is M phi_prev, and the new source is that one grown by `growth` plus `noise`
times a fresh field, as between two time steps.

Case fields (all cases): kind, n, levels, degree, precision ("mixed", "fp64",
"fp32"), smoother, alpha, box (box length, h = box / n), power and cut
(source spectrum k^power exp(-(k / (cut n 2 pi))^2)), growth, noise.
Kinds:
  solve    one solve to `tol` with a context the program keeps, warm if
           `warm`; mesh: 0 seven-point, else the 19-point operator
  pcg      the same with multigrid-preconditioned conjugate gradients
  pm_step  growth-scaled guess, `cycles` warm cycles, force in float32
  mesh_step  geometry of a new deformation, a new context on it, a warm solve
           (to `tol`, or `cycles` cycles where that is not 0), force
  grad     loss sum(w phi) through geometry, source and solve, and its
           gradients with respect to the deformation and the source field
"""
import math

import torch

import paper_2607_10983_amd as mgpu

TWO_PI = 2.0 * math.pi
PAIRS = ((0, 1, 3), (0, 2, 4), (1, 2, 5))  # (a, b, stored component)


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def _case(kind, n, **kw):
    c = {"kind": kind, "n": n, "levels": n.bit_length() - 2, "degree": 3, "precision": "mixed",
         "smoother": "chebyshev", "alpha": 8.0, "box": 1.0, "power": -1.0, "cut": 0.25, "growth": 1.05,
         "noise": 0.02, "tol": 1e-10, "cycles": 0, "warm": True, "mesh": 0.0, "psi_levels": False}
    c.update(kw)
    return c


def listed():
    return [
        # small calls, where launches and latency count: a unit-box test problem solved from zero
        _case("solve", 32, name="flat_32_mixed_cold", levels=4, warm=False),
        # the same in plain float64 with the 16^3 coarsest level and degree 4 of larger runs
        _case("solve", 64, name="flat_64_fp64_warm", levels=3, degree=4, precision="fp64"),
        # a time step of a particle-mesh run in single precision: few warm cycles, then the force
        _case("pm_step", 128, name="pm_128_fp32_step", precision="fp32", cycles=4),
        # the benchmark's solve: 256^3, warm, mixed precision, to 1e-10
        _case("solve", 256, name="flat_256_mixed_warm", cut=0.0),
        # Krylov variant in float64 for the same problem
        _case("pcg", 256, name="flat_256_fp64_pcg", precision="fp64", cut=0.0),
        # one GPU's share of a large run: four warm cycles and the force of a 512^3 step
        _case("pm_step", 512, name="pm_512_mixed_step", levels=6, degree=4, cycles=4),
        # the largest grid that the benchmark runs, two warm cycles
        _case("pm_step", 1024, name="pm_1024_mixed_step", levels=7, degree=4, cycles=2),
        # a whole moving-mesh step on a small grid: geometry, new context, solve, force
        _case("mesh_step", 64, name="mesh_64_mixed_step", mesh=0.6),
        # repeated solves on one mesh (several sources, or an adjoint) at full size
        _case("solve", 256, name="mesh_256_mixed_warm", mesh=0.6),
        # the same in plain float64 on a medium grid, levels rediscretised from the deformation
        _case("solve", 128, name="mesh_128_fp64_warm", mesh=0.6, precision="fp64", psi_levels=True),
        # gradient of a loss through geometry, source and solve: one training or inference step
        _case("grad", 128, name="mesh_128_mixed_grad", mesh=0.6),
        # moving-mesh step with the weighted-Jacobi setting: two sweeps, six warm cycles
        _case("mesh_step", 256, name="mesh_256_jacobi_step", mesh=0.6, smoother="jacobi", cycles=6, psi_levels=True),
    ]


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    while True:
        kind = rng.choice(("solve", "solve", "pm_step", "pm_step", "pcg", "mesh_solve", "mesh_solve", "mesh_step",
                           "grad"))
        mesh = 0.0
        if kind in ("mesh_solve", "mesh_step", "grad"):
            n = 2 ** rng.randint(4, 7 if kind == "grad" else 8)
            mesh = round(rng.uniform(0.2, 0.7), 3)
        else:
            n = 2 ** rng.randint(4, 9)
        # the coarsest level has 4^3, 8^3 or (seven-point) 16^3 points
        coarsest = rng.choice((4, 4, 8) if mesh else (4, 4, 8, 16))
        coarsest = min(coarsest, n // 2)
        c = _case("solve" if kind == "mesh_solve" else kind, n, mesh=mesh,
                  levels=int(math.log2(n // coarsest)) + 1,
                  degree=rng.choice((2, 3, 3, 4, 5)),
                  precision=rng.choice(("mixed", "mixed", "fp64")),
                  alpha=round(rng.uniform(5.0, 12.0), 3),
                  box=rng.choice((1.0, round(10.0 ** rng.uniform(0.0, 3.0), 3))),
                  power=round(rng.uniform(-1.5, -0.5), 3),
                  cut=rng.choice((0.0, round(rng.uniform(0.15, 0.35), 3))),
                  growth=round(rng.uniform(1.01, 1.1), 4),
                  noise=round(10.0 ** rng.uniform(-2.3, -1.3), 4),
                  tol=float("%.2g" % 10.0 ** rng.uniform(-10.3, -9.0)),
                  warm=rng.random() < 0.75)
        if kind == "pm_step":
            c["cycles"] = rng.randint(2, 4)
            if rng.random() < 0.3:
                c["precision"] = "fp32"
        if mesh:
            c["psi_levels"] = kind != "grad" and rng.random() < 0.4
            if kind != "grad" and rng.random() < 0.25:
                c["smoother"] = "jacobi"
                c["cycles"] = rng.randint(4, 8) if kind == "mesh_step" else 0
        if work(c)["bytes"] <= most:
            return c


def work(case):
    """One pass: per V-cycle the potential and the source are read and the
    potential is written, in double (24 bytes a point), and the coefficients
    are read once; a step adds its geometry, guess and force.  Operations: the
    operator's, as often as the smoothing passes and the two residuals apply it."""
    n3 = float(case["n"]) ** 3
    mesh = case["mesh"] > 0.0
    cycles = case["cycles"] or math.ceil(-math.log10(case["tol"]) * (1.2 if mesh else 1.0))
    if case["kind"] == "pcg":
        cycles = math.ceil(0.75 * cycles)
    coeff = 6.0 * (8 if case["precision"] == "fp64" else 4) if mesh else 0.0
    applications = (2 * (2 if case["smoother"] == "jacobi" else case["degree"]) + 2) * 8.0 / 7.0
    cycle_bytes = 24.0 + coeff
    cycle_flops = applications * (120.0 if mesh else 12.0)
    by, fl = cycles * cycle_bytes, cycles * cycle_flops
    if case["kind"] == "pm_step":
        by += 8 + 8 + 8 + 12  # guess read and written, force
        fl += 25
    if case["kind"] == "mesh_step":
        by += 8 + coeff + 8 + 16 + 12  # deformation -> coefficients and volume; force
        fl += 160
    if case["kind"] == "grad":
        by, fl = 2 * by + 2 * (8 + coeff + 8) + 16, 2 * fl + 600
    return {"bytes": by * n3, "flops": fl * n3}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _freqs(n, dev):
    m = torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device=dev)
    mr = torch.fft.rfftfreq(n, d=1.0 / n, dtype=torch.float64, device=dev)
    return m[:, None, None], m[None, :, None], mr[None, None, :]


def _field(n, seed, power, cut, dev):
    """Zero-mean unit-variance Gaussian random field of spectrum
    k^power exp(-(k/cut)^2) (frequencies in cycles per box, no cutoff when 0)."""
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    w = torch.randn((n, n, n), generator=g, dtype=torch.float64, device=dev)
    W = torch.fft.rfftn(w)
    del w
    z, y, x = _freqs(n, dev)
    k2 = z * z + y * y + x * x
    k2[0, 0, 0] = 1.0
    W *= k2 ** (0.25 * power)
    if cut > 0:
        W *= torch.exp(-0.5 * k2 / (cut * cut))
    del k2
    W[0, 0, 0] = 0.0
    f = torch.fft.irfftn(W, s=(n, n, n))
    del W
    f -= f.mean()
    f /= f.square().mean().sqrt()
    return f


def _eig(n, h, dev):
    m, _, mr = _freqs(n, dev)
    s, sr = torch.sin(math.pi * m / n) ** 2, torch.sin(math.pi * mr / n) ** 2
    return -(4.0 / (h * h)) * (s + s.reshape(1, n, 1) + sr)


def _flat_inverse(b, h):
    n = b.shape[0]
    lam = _eig(n, h, b.device)
    lam[0, 0, 0] = 1.0
    B = torch.fft.rfftn(b)
    B /= lam
    B[0, 0, 0] = 0.0
    del lam
    return torch.fft.irfftn(B, s=b.shape)


def _inputs(case, seed):
    """(psi or None, the coefficients the context gets or None, phi_prev, b)."""
    dev = torch.device("cuda")
    n, h, s = case["n"], case["box"] / case["n"], 16 * int(seed)
    cut = case["cut"] * n
    psi = None
    if case["mesh"] > 0.0:
        psi = _field(n, s + 1, -4.0, min(16.0, n / 8.0), dev)
        H = _hessian(psi, h)
        rows = [sum(H[COMP[a][b]].abs() for b in range(3)) for a in range(3)]
        # row sums of |mesh * Hess| at most `mesh`, so I + Hess psi is positive definite everywhere
        psi *= case["mesh"] / max(float(r.max()) for r in rows)
        del H, rows
    src = _field(n, s + 2, case["power"], cut, dev)
    phi_prev = _flat_inverse(src, h)
    eta = _field(n, s + 3, case["power"], cut, dev)
    return psi, src, phi_prev, eta


def _sources(case, psi, C, src, phi_prev, eta):
    h = case["box"] / case["n"]
    if psi is None:
        return case["growth"] * src + case["noise"] * eta
    return case["growth"] * _apply_var(phi_prev, C, h) + case["noise"] * eta


def _opts(case):
    o = {"levels": case["levels"], "degree": case["degree"], "precision": case["precision"], "alpha": case["alpha"],
         "h": case["box"] / case["n"]}
    if case["smoother"] == "jacobi":
        o["smoother"] = "jacobi"
    return o


def prepare(case, seed):
    psi, src, phi_prev, eta = _inputs(case, seed)
    n, h = case["n"], case["box"] / case["n"]
    st = {"case": case, "h": h, "psi": psi, "opts": _opts(case)}
    if case["kind"] in ("solve", "pcg", "pm_step"):
        C = None
        if psi is not None:
            C = _geometry(psi, h)[0]
            if not case["psi_levels"] and case["precision"] == "mixed":
                C = C.float()  # the coefficients as a program with float32 storage hands them over
        st["b"] = _sources(case, psi, None if C is None else C.double(), src, phi_prev, eta)
        st["phi_prev"] = phi_prev if case["warm"] or case["kind"] == "pm_step" else None
        st["mg"] = mgpu.Multigrid(n, **st["opts"]) if psi is None else (
            mgpu.Multigrid(n, psi=psi, **st["opts"]) if case["psi_levels"] else
            mgpu.Multigrid(n, coeff=C, **st["opts"]))
    elif case["kind"] == "mesh_step":
        st["b"] = _sources(case, psi, _geometry(psi, h)[0], src, phi_prev, eta)
        st["phi_prev"] = phi_prev
    else:  # grad: the density contrast and the loss weight
        st["g"], st["w"] = src, eta
    torch.cuda.synchronize()
    return st


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "solve":
        phi, info = st["mg"].solve(st["b"], phi0=st["phi_prev"], tol=c["tol"], max_cycles=100)
        return {"phi": phi, "cycles": info.cycles}
    if kind == "pcg":
        phi, info = st["mg"].solve_pcg(st["b"], phi0=st["phi_prev"], tol=c["tol"], max_iter=100)
        return {"phi": phi, "iterations": info.cycles}
    if kind == "pm_step":
        phi = mgpu.predict("growth", [st["phi_prev"]], growth=c["growth"])
        st["mg"].cycles(phi, st["b"], c["cycles"])
        return {"phi": phi, "force": mgpu.accel(phi, scale=0.45, h=st["h"], dtype=torch.float32)}
    if kind == "mesh_step":
        dt = torch.float64 if c["precision"] == "fp64" else torch.float32
        if c["psi_levels"]:
            mg = mgpu.Multigrid(c["n"], psi=st["psi"], **st["opts"])
        else:
            C, _ = mgpu.geometry(st["psi"], h=st["h"], dtype=dt)
            mg = mgpu.Multigrid(c["n"], coeff=C, **st["opts"])
        out = {}
        if c["cycles"]:
            phi = mgpu.predict("growth", [st["phi_prev"]], growth=c["growth"])
            mg.cycles(phi, st["b"], c["cycles"])
        else:
            phi, info = mg.solve(st["b"], phi0=st["phi_prev"], tol=c["tol"], max_cycles=100)
            out["cycles"] = info.cycles
        mg.close()
        return {"phi": phi, "force": mgpu.accel(phi, st["psi"], scale=0.45, h=st["h"], dtype=torch.float32), **out}
    psi = st["psi"].clone().requires_grad_(True)
    g = st["g"].clone().requires_grad_(True)
    C, sg = mgpu.geometry_fn(psi, h=st["h"])
    b = sg * (g - (g * sg).sum() / sg.sum())
    opts = {k: v for k, v in st["opts"].items()}
    phi = mgpu.solve(b, C, tol=c["tol"], max_cycles=100, **opts)
    loss = (st["w"] * phi).sum()
    dpsi, dg = torch.autograd.grad(loss, (psi, g))
    return {"phi": phi.detach(), "dpsi": dpsi, "dg": dg}


# ---------------------------------------------------------------------------
# The same in plain float64 torch, one shifted copy per stencil leg
# ---------------------------------------------------------------------------

COMP = ((0, 3, 4), (3, 1, 5), (4, 5, 2))


def _sh(u, a, s):
    """out[i] = u[i + s e_a], direction 0 = x (the last axis)."""
    return torch.roll(u, -s, dims=2 - a)


def _hessian(psi, h):
    H = [(_sh(psi, a, 1) - 2.0 * psi + _sh(psi, a, -1)) / (h * h) for a in range(3)]
    for a, b, _ in PAIRS:
        p, m = _sh(psi, a, 1), _sh(psi, a, -1)
        H.append((_sh(p, b, 1) - _sh(p, b, -1) - _sh(m, b, 1) + _sh(m, b, -1)) / (4.0 * h * h))
    return H


def _inverse3(J):
    """Determinant and inverse of the symmetric matrices stored as six fields."""
    xx, yy, zz, xy, xz, yz = J
    k = [yy * zz - yz * yz, xx * zz - xz * xz, xx * yy - xy * xy, xz * yz - xy * zz, xy * yz - xz * yy,
         xy * xz - yz * xx]
    det = xx * k[0] + xy * k[3] + xz * k[4]
    return det, [v / det for v in k]


def _geometry(psi, h):
    """(C, sqrt g): C = det(J) J^-1 J^-1 with J = I + Hess psi, as (6, n, n, n)."""
    H = _hessian(psi, h)
    det, K = _inverse3([H[0] + 1.0, H[1] + 1.0, H[2] + 1.0] + H[3:])
    C = [None] * 6
    for a in range(3):
        for b in range(a, 3):
            C[COMP[a][b]] = det * sum(K[COMP[a][j]] * K[COMP[j][b]] for j in range(3))
    return torch.stack(C), det


def _apply_flat(u, h):
    out = -6.0 * u
    for a in range(3):
        out = out + _sh(u, a, 1) + _sh(u, a, -1)
    return out / (h * h)


def _apply_var(u, C, h):
    out = torch.zeros_like(u)
    for a in range(3):
        flux = 0.5 * (C[a] + _sh(C[a], a, 1)) * (_sh(u, a, 1) - u)
        out = out + flux - _sh(flux, a, -1)
    for a, b, c in PAIRS:
        for p, q in ((a, b), (b, a)):
            f = C[c] * (_sh(u, q, 1) - _sh(u, q, -1))
            out = out + 0.25 * (_sh(f, p, 1) - _sh(f, p, -1))
    return out / (h * h)


def _restrict(r):
    for ax in range(3):
        r = 0.25 * torch.roll(r, 1, dims=ax) + 0.5 * r + 0.25 * torch.roll(r, -1, dims=ax)
    return r[::2, ::2, ::2].contiguous()


def _prolong(e):
    for ax in range(3):
        e = torch.stack((e, 0.5 * (e + torch.roll(e, -1, dims=ax))), dim=ax + 1).flatten(ax, ax + 1)
    return e


class _Plain:
    """The cycle of the case in float64: one level per entry of `lev`."""

    def __init__(self, case, C, psi):
        h = case["box"] / case["n"]
        self.case, self.lev = case, []
        for l in range(case["levels"]):
            hl, last = h * 2 ** l, l == case["levels"] - 1
            if C is None:
                self.lev.append((hl, None, 1.0 / (-6.0 / (hl * hl)), 2.0))
                continue
            face = sum(C[a] + 0.5 * (_sh(C[a], a, 1) + _sh(C[a], a, -1)) for a in range(3))
            edge = sum(0.25 * (_sh(C[c], a, sa) + _sh(C[c], b, sb)).abs()
                       for a, b, c in PAIRS for sa in (1, -1) for sb in (1, -1))
            self.lev.append((hl, C, -(hl * hl) / face, float((1.0 + (face + edge) / face).max())))
            if not last and case["psi_levels"]:
                psi = _restrict(psi)
                C = _geometry(psi, 2.0 * hl)[0]
            elif not last:
                C = torch.stack([_restrict(C[c]) for c in range(6)])
        hl, C, _, _ = self.lev[-1]
        self.pinv = None
        if C is not None:
            m = C.shape[1]
            cols = torch.eye(m ** 3, dtype=torch.float64, device=C.device).reshape(-1, m, m, m)
            A = torch.stack([_apply_var(v, C, hl).reshape(-1) for v in cols])
            self.pinv = torch.linalg.pinv(A.cpu(), rtol=1e-10, hermitian=True).to(C.device)

    def apply(self, l, u):
        h, C = self.lev[l][:2]
        return _apply_flat(u, h) if C is None else _apply_var(u, C, h)

    def smooth(self, l, x, b):
        _, _, dinv, lmax = self.lev[l]
        if self.case["smoother"] == "jacobi":
            for _ in range(2):
                x = x + (2.0 / 3.0) * dinv * (b - self.apply(l, x))
            return x
        lmin = lmax / self.case["alpha"]
        theta, delta = 0.5 * (lmax + lmin), 0.5 * (lmax - lmin)
        rho = delta / theta
        d = dinv * (b - self.apply(l, x)) / theta
        x = x + d
        for _ in range(1, self.case["degree"]):
            new = 1.0 / (2.0 * theta / delta - rho)
            d = new * rho * d + (2.0 * new / delta) * (dinv * (b - self.apply(l, x)))
            x = x + d
            rho = new
        return x

    def cycle(self, l, x, b):
        if l == len(self.lev) - 1:
            if self.pinv is None:
                return _flat_inverse(b, self.lev[l][0])
            return (self.pinv @ b.reshape(-1)).reshape(b.shape)
        x = self.smooth(l, x, b)
        e = self.cycle(l + 1, torch.zeros_like(b[::2, ::2, ::2]), _restrict(b - self.apply(l, x)))
        return self.smooth(l, x + _prolong(e), b)

    def cycles(self, x, b, count):
        b = b - b.mean()
        for _ in range(count):
            x = self.cycle(0, x, b)
        return x - x.mean()

    def solve(self, b, x):
        """Cycles until the residual stops falling at its rounding floor."""
        b = b - b.mean()
        x = torch.zeros_like(b) if x is None else x
        last = math.inf
        for _ in range(60):
            x = self.cycle(0, x, b)
            r = float((b - self.apply(0, x)).norm() / b.norm())
            if r > 0.5 * last and r < 1e-11:
                break
            last = r
        return x - x.mean()


def _force(phi, psi, h, scale):
    out = []
    for a in range(3):
        g = _sh(phi, a, -2) - 8.0 * _sh(phi, a, -1)
        g += 8.0 * _sh(phi, a, 1)
        g -= _sh(phi, a, 2)
        out.append(g * (-scale / (12.0 * h)))
    if psi is not None:
        H = _hessian(psi, h)
        _, K = _inverse3([H[0] + 1.0, H[1] + 1.0, H[2] + 1.0] + H[3:])
        out = [sum(K[COMP[a][j]] * out[j] for j in range(3)) for a in range(3)]
    return torch.stack(out)


def exact(case, seed):
    psi, src, phi_prev, eta = _inputs(case, seed)
    n, h, kind = case["n"], case["box"] / case["n"], case["kind"]
    if kind == "grad":
        p, g = psi.clone().requires_grad_(True), src.clone().requires_grad_(True)
        C, sg = _geometry(p, h)
        b = sg * (g - (g * sg).sum() / sg.sum())
        plain = _Plain(case, C.detach(), psi)
        phi, lam = plain.solve(b.detach(), None), plain.solve(eta, None)
        # d(w . M^+ b) = lam . (db - dM phi) with lam = M^+ w
        dpsi, dg = torch.autograd.grad((lam * (b - _apply_var(phi, C, h))).sum(), (p, g))
        return {"phi": phi, "dpsi": dpsi, "dg": dg}
    C = None
    if psi is not None:
        C = _geometry(psi, h)[0]
        if kind != "mesh_step" and not case["psi_levels"] and case["precision"] == "mixed":
            C = C.float().double()
    b = _sources(case, psi, C, src, phi_prev, eta)
    del src, eta
    if kind in ("solve", "pcg") and psi is None:
        return {"phi": _flat_inverse(b, h)}
    plain = _Plain(case, C, psi)
    if case["cycles"]:
        phi = plain.cycles(case["growth"] * phi_prev, b, case["cycles"])
    else:
        phi = plain.solve(b, phi_prev)
    if kind in ("solve", "pcg"):
        return {"phi": phi}
    del plain, b
    return {"phi": phi, "force": _force(phi, psi, h, 0.45)}
