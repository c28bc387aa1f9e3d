"""Cases that time the framework through its public entry points.

Each case is one call of a user's program on inputs that are already on the GPU (or, for the
small dense problem, in host memory, as that call takes them).  The kinds follow a block
iteration from its parts to the whole:

* ``vcycle``:  the geometric multigrid V-cycle of the edge operator, ``Solver.apply("EDGE_VCYCLE")``;
* ``project``: the null-space projection with its nodal multigrid, ``Solver.apply("PROJECT")``;
* ``eigres``:  the eigen-residual of a block, ``Solver.apply("EIGRES")``;
* ``rr``:      the Rayleigh-Ritz products S^* M S and S^* A S, ``Solver.rr_products``;
* ``ritz``:    the small generalised eigenproblem of the Ritz step, ``Solver.ritz_small``;
* ``solve``:   eigenvalues along Bloch parameters, ``Solver.solve_k`` / ``Solver.solve_path``;
* ``batch``:   independent problems of several mesh sizes in one ``Batch.run``.

Sizes come from the configurations in ``synth`` and the workloads of ``bench.py``: 32 x 32 to
1024 x 1024 cells, blocks of 8 to 48 vectors, FP64 and mixed precision.
"""
import math

import numpy as np
import torch

from paper_2304_00337_amd import api

MU = 20.0   # shift of the preconditioned operator: the default's value for the unit cell


def listed():
    return [
        # the preconditioner of the 1024 x 1024 band path (mixed precision): the columns that
        # soft locking leaves of its 48-vector block on average
        dict(name="vcycle 1024 fp32", kind="vcycle", n=1024, m=1024, b=1.0, mixed=True, cols=24),
        # the preconditioner of the 256 x 256 lattice path in plain FP64, all 16 + 8 columns
        dict(name="vcycle 256 fp64", kind="vcycle", n=256, m=256, b=1.0, mixed=False, cols=24),
        # a rectangular cell whose mesh fills no tile evenly, with an odd column count
        dict(name="vcycle 480x288 fp32", kind="vcycle", n=480, m=288, b=0.7, mixed=True, cols=7),
        # the null-space elimination of the 48 start vectors of a 1024 x 1024 point
        dict(name="project 1024 mixed", kind="project", n=1024, m=1024, b=1.0, mixed=True, cols=48),
        # the same for the 2 x 24 basis vectors of an iteration on the 256 x 256 path
        dict(name="project 256 fp64", kind="project", n=256, m=256, b=1.0, mixed=False, cols=48),
        # Ritz-step products at 1024 x 1024: 48 vectors and 36 preconditioned directions
        dict(name="rr 1024 q84", kind="rr", n=1024, m=1024, b=1.0, q=84),
        # the Ritz step's dense problem on the 256 x 256 path (24 of 48) and on the 1024 x 1024
        # path (48 of 84)
        dict(name="ritz q48", kind="ritz", q=48, want=24),
        dict(name="ritz q84", kind="ritz", q=84, want=48),
        # the smallest call in use: one Bloch parameter on a 32 x 32 mesh, latency and launches
        dict(name="point 32 fp64", kind="solve", n=32, m=32, b=1.0, mixed=False, field=False, nev=8, nthrow=4,
             points=1, nested=False, tol=1e-8),
        # three points of the 256 x 256 lattice path, the later ones extrapolated
        dict(name="path 256 fp64", kind="solve", n=256, m=256, b=1.0, mixed=False, field=False, nev=16, nthrow=8,
             points=3, nested=False, tol=1e-8),
        # many small problems at once, as a parameter study submits them
        dict(name="batch 64-192 mixed", kind="batch", n=64, count=9, mixed=True, nev=8, nthrow=4, tol=1e-8),
        # a first point of the 1024 x 1024 path: random two-phase medium, nested start, soft locking
        dict(name="point 1024 mixed", kind="solve", n=1024, m=1024, b=1.0, mixed=True, field=True, nev=32, nthrow=16,
             points=1, nested=True, tol=1e-6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mesh(rng, lo, hi):
    """n0 2^l cells with n0 in 8..15, as a mesh that coarsens to a small direct solve has."""
    n = _log_int(rng, lo, hi)
    l = max(0, n.bit_length() - 4)
    return min(max(n >> l, 8), 15) << l


def _pair(rng, lo, hi):
    n = _mesh(rng, lo, hi)
    l = max(0, n.bit_length() - 4)
    return n, rng.randint(8, 15) << l   # same depth: the hierarchy reaches 8..15 in both directions


def draw(rng):
    kind = rng.choice(["vcycle", "vcycle", "project", "project", "eigres", "rr", "ritz", "solve", "batch"])
    mixed = rng.random() < 0.6
    aspect = rng.choice([1.0, 1.0, 0.7, round(rng.uniform(0.5, 1.6), 3)])
    if kind in ("vcycle", "project", "eigres"):
        n, m = _pair(rng, 32, 1000)
        cols = _log_int(rng, 1, 48 if n * m < 700_000 else 32)
        return dict(kind=kind, n=n, m=m, b=aspect, mixed=mixed, cols=cols)
    if kind == "rr":
        n, m = _pair(rng, 32, 1000)
        return dict(kind=kind, n=n, m=m, b=aspect, q=_log_int(rng, 8, 96))
    if kind == "ritz":
        q = rng.randint(8, 112)
        return dict(kind=kind, q=q, want=max(1, int(q * rng.uniform(0.3, 0.6))))
    if kind == "solve":
        n = _mesh(rng, 32, 512)
        nev = rng.randint(4, 24)
        nested = rng.random() < 0.5 and n >= 64
        return dict(kind=kind, n=n, m=n, b=1.0, mixed=mixed, field=rng.random() < 0.5, nev=nev,
                    nthrow=max(3, nev // 2), points=rng.randint(1, 3), nested=nested, tol=1e-6 if mixed else 1e-8)
    return dict(kind="batch", n=rng.choice([32, 48, 64, 80]), count=rng.randint(3, 12), mixed=mixed,
                nev=rng.randint(4, 12), nthrow=rng.randint(3, 6), tol=1e-8)


# ---- inputs ----------------------------------------------------------------------------------

def _lattice_eps(n, m, rng):
    """One centred disc per cell: radius and contrast of the lattice workloads."""
    r, inside = rng.uniform(0.2, 0.35), rng.uniform(8.0, 12.5)
    x, y = np.meshgrid((np.arange(n) + 0.5) / n - 0.5, (np.arange(m) + 0.5) / m - 0.5)
    return np.where(x * x + y * y <= r * r, inside, 1.0).reshape(-1)


def _field_eps(n, m, rng):
    """Two-phase medium: blurred Gaussian noise above or below zero."""
    fx, fy = np.meshgrid(np.fft.fftfreq(n, 1.0 / n), np.fft.fftfreq(m, 1.0 / m))
    blur = np.exp(-2.0 * (math.pi * 0.05) ** 2 * (fx * fx + fy * fy))
    smooth = np.fft.ifft2(np.fft.fft2(rng.standard_normal((m, n))) * blur).real
    return np.where(smooth > 0, 11.4, 1.0).reshape(-1)


def _bloch(case, rng):
    return (math.pi * rng.uniform(0.2, 0.9), math.pi / case["b"] * rng.uniform(0.1, 0.8))


def _waves(case, k, cols, seed, rough):
    """Smooth divergence-free Bloch fields (random transverse discrete plane waves, as converged
    eigenvectors are), plus `rough` times white noise; complex (cols, 2, m, n) on the GPU."""
    n, m, b = case["n"], case["m"], case["b"]
    gen = torch.Generator("cuda").manual_seed(seed)
    g = min(12, n // 4, m // 4)
    i = torch.arange(-g, g + 1, device="cuda", dtype=torch.float64)
    t1 = ((k[0] + 2 * math.pi * i) / n)[None, :]
    t2 = ((k[1] + 2 * math.pi / b * i) * b / m)[:, None]
    mx, my = (b / m) * n, m / (b * n)
    cx = torch.conj(torch.exp(1j * t2) - 1) * my * (1 - 2 / 3 * torch.sin(t1 / 2) ** 2)
    cy = -torch.conj(torch.exp(1j * t1) - 1) * mx * (1 - 2 / 3 * torch.sin(t2 / 2) ** 2)
    norm = torch.sqrt(abs(cx) ** 2 + abs(cy) ** 2)
    shape = (cols, 2 * g + 1, 2 * g + 1, 2)
    amp = torch.view_as_complex(torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64))
    amp = amp / (norm * (1.0 + i[None, :] ** 2 + i[:, None] ** 2))
    idx = i.long()
    spec = torch.zeros((cols, 2, m, n), dtype=torch.complex128, device="cuda")
    for comp, c in ((0, cx), (1, cy)):
        spec[:, comp, (idx % m)[:, None], (idx % n)[None, :]] = amp * c
    e = torch.fft.ifft2(spec) * (n * m)
    px = torch.exp(1j * k[0] / n * torch.arange(n, device="cuda", dtype=torch.float64))
    py = torch.exp(1j * k[1] * b / m * torch.arange(m, device="cuda", dtype=torch.float64))
    e = e * px * py[:, None]
    if rough:
        for j in range(cols):
            z = torch.randn((2, m, n, 2), generator=gen, device="cuda", dtype=torch.float64)
            e[j] += rough * torch.view_as_complex(z)
    return e


def _planar(e, dtype=torch.float64):
    """complex (cols, 2, m, n) -> planar column block (cols, 2, 2 n m)."""
    flat = e.reshape(e.shape[0], -1)
    return torch.stack([flat.real, flat.imag], dim=1).to(dtype).contiguous()


def _fields(t, m, n):
    """Planar column block -> complex128 (cols, 2, m, n)."""
    t = t.double()
    return torch.complex(t[:, 0], t[:, 1]).reshape(t.shape[0], 2, m, n)


def _block_inputs(case, seed):
    """Permittivity, Bloch parameter and input block of the operator cases."""
    rng = np.random.default_rng(seed)
    n, m = case["n"], case["m"]
    eps = _field_eps(n, m, rng) if min(n, m) >= 256 else _lattice_eps(n, m, rng)
    k = _bloch(case, rng)
    kind = case["kind"]
    cols = case["q"] if kind == "rr" else case["cols"]
    e = _waves(case, k, cols, seed, 1e-3 if kind in ("vcycle", "eigres") else 0.1)
    lam = None
    if kind in ("vcycle", "eigres"):
        lam = torch.tensor(np.sort(rng.uniform(2.0, 150.0, cols)), device="cuda")
    if kind == "vcycle":   # the iteration's residual A e - lambda M e, scaled to unit size
        for j in range(cols):
            op = _Level(n, m, 1.0, case["b"], k, _kappa(eps, n, m))
            r = op.A(e[j:j + 1]) - lam[j] * op.M(e[j:j + 1])
            e[j] = r[0] / r.abs().square().mean().sqrt()
        lam = None
    prec = torch.float32 if case.get("mixed") and kind in ("vcycle", "eigres") else torch.float64
    return eps, k, _planar(e, prec), lam


def _ritz_inputs(case, seed):
    """G and H of a basis [E, C]: `want` nearly orthonormal Ritz vectors and small correction
    directions, for a known spectrum with separated values."""
    q, want = case["q"], case["want"]
    rng = np.random.default_rng(seed)
    lam = 4.0 * (1.0 + np.arange(q) + 0.3 * rng.uniform(-1, 1, q)) * (1.0 + np.arange(q) / q)
    t = 0.02 * (rng.standard_normal((q, q)) + 1j * rng.standard_normal((q, q))) / math.sqrt(q)
    t[:, :want] += np.eye(q)[:, :want]
    c = np.eye(q)[:, want:] + 0.3 * (rng.standard_normal((q, q - want)) + 1j * rng.standard_normal((q, q - want))) / math.sqrt(q)
    t[:, want:] = (t[:, want:] + c) * 10.0 ** rng.uniform(-4, -1, q - want)
    g = t.conj().T @ t
    h = t.conj().T @ (lam[:, None] * t)
    return 0.5 * (g + g.conj().T), 0.5 * (h + h.conj().T)


def _random_block(p, ne, seed):
    gen = torch.Generator("cuda").manual_seed(seed)
    return torch.randn((p, 2, ne), generator=gen, device="cuda", dtype=torch.float64) / math.sqrt(2.0)


def _solve_inputs(case, seed):
    rng = np.random.default_rng(seed)
    n, m = case["n"], case["m"]
    eps = _field_eps(n, m, rng) if case["field"] else _lattice_eps(n, m, rng)
    k1 = math.pi * rng.uniform(0.3, 0.5)
    ks = np.array([(k1 + 0.1 * math.pi * t, 0.2 * math.pi) for t in range(case["points"])])
    return eps, ks


def prepare(case, seed):
    kind, prec = case["kind"], "mixed" if case.get("mixed") else "fp64"
    if kind == "ritz":
        g, h = _ritz_inputs(case, seed)
        solver = api.Solver(16, 16, 1.0, 1.0, np.ones(256), nev=4)
        return dict(kind=kind, solver=solver, g=g, h=h, want=case["want"])
    if kind == "solve":
        eps, ks = _solve_inputs(case, seed)
        n, m, p = case["n"], case["m"], case["nev"] + case["nthrow"]
        opts = dict(nested_start=1, lock_rel=1.0, throw_precond=4) if case["nested"] else {}
        solver = api.Solver(n, m, 1.0, case["b"], eps, nev=case["nev"], nthrow=case["nthrow"], precision=prec,
                            tol=case["tol"], tol_floor=1, max_iter=300, **opts)
        start = None if case["nested"] else _random_block(p, 2 * n * m, seed)
        return dict(kind=kind, solver=solver, ks=ks, start=start)
    if kind == "batch":
        problems = []
        rng = np.random.default_rng(seed)
        for i in range(case["count"]):
            n = case["n"] * (i % 3 + 1)   # three mesh sizes in turn
            problems.append(dict(n=n, m=n, a=1.0, b=1.0, eps=_lattice_eps(n, n, rng), nev=case["nev"],
                                 nthrow=case["nthrow"], ks=np.array([rng.uniform(0.2, 0.9, 2) * math.pi]),
                                 start=_random_block(case["nev"] + case["nthrow"], 2 * n * n, seed + 100 * i)))
        batch = api.Batch(precision=prec, tol=case["tol"], tol_floor=1, max_iter=300)
        return dict(kind=kind, batch=batch, problems=problems)
    eps, k, x, lam = _block_inputs(case, seed)
    cols = x.shape[0]
    p = -(-cols // 3) if kind in ("project", "rr") else cols   # a handle takes 3 p basis columns
    solver = api.Solver(case["n"], case["m"], 1.0, case["b"], eps, nev=p, nthrow=0, precision=prec, mu=MU)
    solver.set_k(*k)
    return dict(kind=kind, solver=solver, x=x, lam=lam, out=torch.empty_like(x))


def run(state):
    kind = state["kind"]
    if kind == "vcycle":
        return state["solver"].apply("EDGE_VCYCLE", state["x"], out=state["out"])
    if kind == "project":
        return state["solver"].apply("PROJECT", state["x"], out=state["out"])
    if kind == "eigres":
        return state["solver"].apply("EIGRES", state["x"], y=state["lam"], out=state["out"])
    if kind == "rr":
        return state["solver"].rr_products(state["x"])
    if kind == "ritz":
        theta, y = state["solver"].ritz_small(state["g"], state["h"], state["want"])
        return theta, _fixed_phase(y)
    if kind == "batch":
        return [dict(evals=r["evals"], converged=r["converged"]) for r in state["batch"].run(state["problems"])]
    solver = state["solver"]
    solver.reset_history()   # every pass starts from the start block or the nested start
    if len(state["ks"]) == 1:
        r = solver.solve_k(*state["ks"][0], start=state["start"], allow_noconv=True)
    else:
        r = solver.solve_path(state["ks"], start=state["start"], allow_noconv=True)
    return dict(evals=r["evals"], converged=r["converged"])


def _fixed_phase(y):
    """The vectors with their free phase fixed: the largest entry of each real and positive."""
    big = y[np.abs(y).argmax(axis=0), np.arange(y.shape[1])]
    return y * (np.abs(big) / big)


# ---- work ------------------------------------------------------------------------------------

def _work_block(kind, nm, cols, size):
    """Bytes and operations of one operator on `cols` columns (size: bytes of a real number)."""
    edge = 2 * 2 * nm * size   # one complex edge vector
    if kind == "vcycle":   # residual in, correction out, coefficient in; two sweeps of patch solves per level
        return 2 * cols * edge + nm * size, cols * nm * (2 * 250 + 130) * 4 / 3
    if kind == "project":   # block in and out; two nodal cycles of two sweeps, L^* M and L
        return 2 * cols * edge, cols * nm * (2 * (2 * 35 + 45) * 4 / 3 + 100)
    if kind == "eigres":
        return 2 * cols * edge + nm * size, cols * nm * 80
    return cols * edge + nm * size + 64 * cols * cols, 4 * cols * cols * 3 * nm   # rr


def work(case):
    kind = case["kind"]
    if kind == "ritz":
        q, w = case["q"], case["want"]
        return dict(bytes=32 * q * q + 16 * q * w + 8 * w, flops=4 * (q ** 3 * 16 / 3 + 4 * q * q * w))
    if kind in ("solve", "batch"):
        sizes = ([(case["n"] * (i % 3 + 1)) ** 2 for i in range(case["count"])] if kind == "batch"
                 else [case["n"] * case["m"]])
        p, steps = case["nev"] + case["nthrow"], 20 * case.get("points", 1)   # a converging run's iterations
        total = dict(bytes=0.0, flops=0.0)
        for nm in sizes:
            parts = [_work_block(k, nm, c, s) for k, c, s in (
                ("eigres", p, 8), ("vcycle", p, 4 if case["mixed"] else 8), ("project", 2 * p, 8), ("rr", 2 * p, 8))]
            total["bytes"] += steps * (sum(b for b, _ in parts) + 3 * p * 32 * nm)   # and S Y: 2 p in, p out
            total["flops"] += steps * (sum(f for _, f in parts) + 8 * 2 * p * p * 2 * nm)
        return total
    cols = case["q"] if kind == "rr" else case["cols"]
    size = 4 if case.get("mixed") and kind in ("vcycle", "eigres") else 8
    bytes_, flops = _work_block(kind, case["n"] * case["m"], cols, size)
    return dict(bytes=bytes_, flops=flops)


# ---- the same values in plain 64-bit torch and numpy --------------------------------------------

def _kappa(eps, n, m):
    return (1.0 / torch.tensor(eps, dtype=torch.float64, device="cuda")).reshape(m, n)


class _Level:
    """One level of the discretisation in complex128: fields are (cols, 2, m, n) for edges
    (x-edges, y-edges) and (cols, m, n) for nodes, extended across the period by Bloch phases."""

    def __init__(self, n, m, a, b, k, kappa):
        self.n, self.m, self.a, self.b, self.k, self.kappa = n, m, a, b, k, kappa
        h1, h2 = a / n, b / m
        self.s, self.mx, self.my = 1.0 / (h1 * h2), h2 / h1, h1 / h2
        self.alpha, self.beta = np.exp(1j * k[0] * a), np.exp(1j * k[1] * b)
        r, q = self.mx, self.my
        self.c0, self.cx, self.cy, self.cd = 4 / 3 * (r + q), -2 / 3 * r + q / 3, r / 3 - 2 / 3 * q, -(r + q) / 6

    def sh(self, u, d1, d2):
        """u at (j1 + d1, j2 + d2)."""
        if d1:
            u = torch.roll(u, -d1, -1)
            if d1 > 0:
                u[..., -1] *= self.alpha
            else:
                u[..., 0] *= self.alpha.conjugate()
        if d2:
            u = torch.roll(u, -d2, -2)
            if d2 > 0:
                u[..., -1, :] *= self.beta
            else:
                u[..., 0, :] *= self.beta.conjugate()
        return u

    def A(self, e):
        x, y = e[:, 0], e[:, 1]
        kw = self.s * self.kappa * (self.sh(x, 0, 1) - x + y - self.sh(y, 1, 0))
        return torch.stack([self.sh(kw, 0, -1) - kw, kw - self.sh(kw, -1, 0)], dim=1)

    def M(self, e):
        x, y = e[:, 0], e[:, 1]
        return torch.stack([self.mx * (2 / 3 * x + (self.sh(x, 0, 1) + self.sh(x, 0, -1)) / 6),
                            self.my * (2 / 3 * y + (self.sh(y, 1, 0) + self.sh(y, -1, 0)) / 6)], dim=1)

    def K(self, e):
        return self.A(e) + MU * self.M(e)

    def L(self, f):
        return torch.stack([self.sh(f, 1, 0) - f, self.sh(f, 0, 1) - f], dim=1)

    def Lh(self, e):
        x, y = e[:, 0], e[:, 1]
        return self.sh(x, -1, 0) - x + self.sh(y, 0, -1) - y

    def P(self, f):
        ex, ey = self.sh(f, 1, 0) + self.sh(f, -1, 0), self.sh(f, 0, 1) + self.sh(f, 0, -1)
        return self.c0 * f + self.cx * ex + self.cy * ey + self.cd * (self.sh(ex, 0, 1) + self.sh(ex, 0, -1))

    def coarser(self):
        kap = self.kappa
        kc = 0.25 * (kap[::2, ::2] + kap[1::2, ::2] + kap[::2, 1::2] + kap[1::2, 1::2])
        return _Level(self.n // 2, self.m // 2, self.a, self.b, self.k, kc)

    def patches(self):
        """Per node the inverse of the 4 x 4 patch system of K over (right, left, upper, lower)
        edge, (4, 4, m, n): the gradient direction apart, on which K is MU times the mass."""
        d = torch.tensor([self.mx, self.mx, self.my, self.my], dtype=torch.float64) * (2 / 3)
        z = torch.sqrt(d) * torch.tensor([-1.0, 1.0, -1.0, 1.0], dtype=torch.float64)
        q = torch.linalg.qr(torch.cat([(z / z.norm())[:, None], torch.eye(4, dtype=torch.float64)], dim=1))[0]
        t = (q / torch.sqrt(d)[:, None]).cuda()
        ne, nw = self.kappa, torch.roll(self.kappa, 1, 1)
        sw, se = torch.roll(nw, 1, 0), torch.roll(ne, 1, 0)
        loc = torch.zeros((self.m, self.n, 4, 4), dtype=torch.float64, device="cuda")
        for kap, c in ((ne, (-1, 0, 1, 0)), (nw, (0, -1, -1, 0)), (sw, (0, 1, 0, -1)), (se, (1, 0, 0, 1))):
            c = torch.tensor(c, dtype=torch.float64, device="cuda")
            loc += self.s * kap[..., None, None] * (c[:, None] * c)
        rest = t[:, 1:]
        s = sum(loc[..., i:i + 1, j:j + 1] * (rest[i][:, None] * rest[j]) for i in range(4) for j in range(4))
        s = torch.linalg.inv((s + MU * torch.eye(3, dtype=torch.float64, device="cuda")).cpu()).cuda()
        w = (t[:, 0][:, None] * t[:, 0]) / MU + sum(
            s[..., i:i + 1, j:j + 1] * (rest[:, i][:, None] * rest[:, j]) for i in range(3) for j in range(3))
        return w.permute(2, 3, 0, 1)


def _only(colour, f):
    """f at the nodes of one colour, zero elsewhere."""
    out = torch.zeros_like(f)
    i, j = colour & 1, colour >> 1
    out[..., j::2, i::2] = f[..., j::2, i::2]
    return out


def _edge_sweep(lv, w, x, b, colours):
    for c in colours:
        r = b - lv.K(x)
        rx, ry = r[:, 0], r[:, 1]
        r4 = (rx, lv.sh(rx, -1, 0), ry, lv.sh(ry, 0, -1))
        d = [_only(c, sum(w[i, j] * r4[j] for j in range(4))) for i in range(4)]
        x = x + torch.stack([d[0] + lv.sh(d[1], 1, 0), d[2] + lv.sh(d[3], 0, 1)], dim=1)
    return x


def _direct(op, b):
    """op^{-1} b on the coarsest level."""
    shape = b.shape
    size = b[0].numel()
    eye = torch.eye(size, dtype=torch.complex128, device="cuda").reshape(size, *shape[1:])
    mat = op(eye).reshape(size, size).T.cpu().numpy()
    x = np.linalg.solve(mat, b.reshape(shape[0], size).T.cpu().numpy())
    return torch.tensor(np.ascontiguousarray(x.T), device="cuda").reshape(shape)


def _coarsens(lv):
    return lv.n % 2 == 0 and lv.m % 2 == 0 and lv.n // 2 >= 8 and lv.m // 2 >= 8


def _edge_vcycle(lv, b):
    if not _coarsens(lv):
        return _direct(lv.K, b)
    w = lv.patches()
    x = _edge_sweep(lv, w, torch.zeros_like(b), b, (0, 1, 2, 3))
    r = b - lv.K(x)
    rx, ry = r[:, 0], r[:, 1]
    rx = 0.5 * rx + 0.25 * (lv.sh(rx, 0, 1) + lv.sh(rx, 0, -1))
    ry = 0.5 * ry + 0.25 * (lv.sh(ry, 1, 0) + lv.sh(ry, -1, 0))
    low = lv.coarser()
    c = _edge_vcycle(low, torch.stack([(rx + lv.sh(rx, 1, 0))[:, ::2, ::2], (ry + lv.sh(ry, 0, 1))[:, ::2, ::2]], 1))
    x[:, 0, ::2] += (0.5 * c[:, 0]).repeat_interleave(2, -1)
    x[:, 0, 1::2] += (0.25 * (c[:, 0] + low.sh(c[:, 0], 0, 1))).repeat_interleave(2, -1)
    x[:, 1, :, ::2] += (0.5 * c[:, 1]).repeat_interleave(2, -2)
    x[:, 1, :, 1::2] += (0.25 * (c[:, 1] + low.sh(c[:, 1], 1, 0))).repeat_interleave(2, -2)
    return _edge_sweep(lv, w, x, b, (3, 2, 1, 0))


def _nodal_vcycle(lv, b):
    if not _coarsens(lv):
        return _direct(lv.P, b)
    x = torch.zeros_like(b)
    for c in (0, 1, 2, 3):
        x = x + _only(c, (b - lv.P(x)) / lv.c0)
    r = b - lv.P(x)
    r = r + 0.5 * (lv.sh(r, 1, 0) + lv.sh(r, -1, 0))
    r = r + 0.5 * (lv.sh(r, 0, 1) + lv.sh(r, 0, -1))
    low = lv.coarser()
    c = _nodal_vcycle(low, r[:, ::2, ::2].contiguous())
    up = 0.5 * (c + low.sh(c, 0, 1))
    x[:, ::2, ::2] += c
    x[:, ::2, 1::2] += 0.5 * (c + low.sh(c, 1, 0))
    x[:, 1::2, ::2] += up
    x[:, 1::2, 1::2] += 0.5 * (up + low.sh(up, 1, 0))
    for c in (3, 2, 1, 0):
        x = x + _only(c, (b - lv.P(x)) / lv.c0)
    return x


def _project(lv, u):
    """u - L phi with phi from two nodal V-cycles, the discrete plane wave of k solved exactly."""
    n, m = lv.n, lv.m
    # (k lies inside the first Brillouin zone here)
    t1, t2 = lv.k[0] * lv.a / n, lv.k[1] * lv.b / m
    wave = torch.exp(1j * t1 * torch.arange(n, device="cuda", dtype=torch.float64)) * torch.exp(
        1j * t2 * torch.arange(m, device="cuda", dtype=torch.float64))[:, None]
    s1, s2 = math.sin(t1 / 2) ** 2, math.sin(t2 / 2) ** 2
    lam = 4 * s1 * lv.mx * (1 - 2 / 3 * s2) + 4 * s2 * lv.my * (1 - 2 / 3 * s1)
    part = lambda f: (wave.conj() * f).mean(dim=(-2, -1), keepdim=True)  # noqa: E731
    b = lv.Lh(lv.M(u))
    c = part(b)
    b = b - c * wave
    phi = _nodal_vcycle(lv, b)
    phi = phi + _nodal_vcycle(lv, b - lv.P(phi))
    return u - lv.L(phi + (c / lam - part(phi)) * wave)


def _dense_spectrum(case, eps, k, nev):
    """The nev smallest non-zero eigenvalues by a dense solve; the gradients are the zeros."""
    n, m = case["n"], case["m"]
    lv = _Level(n, m, 1.0, case["b"], k, _kappa(eps, n, m))
    eye = torch.eye(2 * n * m, dtype=torch.complex128, device="cuda").reshape(-1, 2, m, n)
    a = lv.A(eye).reshape(2 * n * m, -1).T.cpu().numpy()
    mass = lv.M(eye).reshape(2 * n * m, -1).T.cpu().numpy()
    c = np.linalg.inv(np.linalg.cholesky(mass))
    v = np.linalg.eigvalsh(c @ a @ c.conj().T)
    return v[n * m:n * m + nev]


def exact(case, seed):
    kind = case["kind"]
    if kind == "ritz":
        g, h = _ritz_inputs(case, seed)
        c = np.linalg.inv(np.linalg.cholesky(g))
        theta, y = np.linalg.eigh(c @ h @ c.conj().T)
        return theta[:case["want"]], _fixed_phase((c.conj().T @ y)[:, :case["want"]])
    if kind == "batch":
        return None
    if kind == "solve":
        if case["n"] * case["m"] > 1100 or case["points"] > 1:
            return None
        eps, ks = _solve_inputs(case, seed)
        return dict(evals=_dense_spectrum(case, eps, tuple(ks[0]), case["nev"]), converged=None)
    eps, k, x, lam = _block_inputs(case, seed)
    n, m = case["n"], case["m"]
    lv = _Level(n, m, 1.0, case["b"], k, _kappa(eps, n, m))
    x = _fields(x, m, n)
    if kind == "rr":
        flat = lambda e: e.reshape(e.shape[0], -1)  # noqa: E731
        return tuple(_conj_product(flat(x), flat(op(x))) for op in (lv.M, lv.A))
    if kind == "eigres":
        return _planar(lv.A(x) - lam[:, None, None, None] * lv.M(x))
    op = _edge_vcycle if kind == "vcycle" else _project
    return torch.cat([_planar(op(lv, x[j:j + 8])) for j in range(0, x.shape[0], 8)])


def _conj_product(a, b):
    """conj(a) b^T for complex (columns, length), in FP64."""
    ar, ai, br, bi = (t.contiguous() for t in (a.real, a.imag, b.real, b.imag))
    re = ar @ br.T + ai @ bi.T
    im = ar @ bi.T - ai @ br.T
    return torch.complex(re, im).cpu().numpy()
