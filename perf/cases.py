"""What a program that uses this library has it do, as cases that can be timed.

A program builds a plan (grid, wavenumber, faces, precision) once, assembles
right-hand sides on the device, solves (one problem or a batch), and may call
the operator and the preconditioner by themselves from a Krylov loop of its
own; the learned correction is evaluated and trained on the same grids.  The
cases below are those calls through `paper_1212_1397_amd.helmholtz6`, on the
grids of the repository's workloads, tests and benchmark and on ragged ones.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1212_1397_amd import helmholtz6 as h6
from paper_1212_1397_amd.workloads import init_net_params

DNS = "DDNNSS"      # x Dirichlet, y Neumann, z Sommerfeld: the benchmark's faces


def listed():
    return [
        # the smallest whole solve (the dirichlet-32 workload's grid, k, restart
        # and tolerance): launches and waits count, not bandwidth
        dict(name="solve-dirichlet-32", kind="solve", nx=32, ny=32, nz=32, bc="DDDDDD", kh=10 / 33, damp=0.0,
             nsrc=1, precision="fp64", method="gmres", restart=20, tol=1e-10),
        # the dns-128 workload in flexible GMRES with the complex64 preconditioner, to the
        # tolerance of the reference solutions that the learned correction trains on
        dict(name="solve-dns-128-mixed", kind="solve", nx=128, ny=128, nz=128, bc=DNS, kh=40 / 129, damp=0.01,
             nsrc=1, precision="mixed", method="fgmres", restart=30, tol=1e-11),
        # bench.py's headline: dns-256, mixed stationary iteration
        dict(name="solve-dns-256-mixed-sks", kind="solve", nx=256, ny=256, nz=256, bc=DNS, kh=80 / 257, damp=0.01,
             nsrc=8, precision="mixed", method="sks", restart=30, tol=1e-8),
        # a grid of the paper's tables (h = 1/256, k = 20) in plain FP64 GMRES
        dict(name="solve-table-255-fp64", kind="solve", nx=255, ny=255, nz=255, bc="DDDDND", kh=20 / 256, damp=0.0,
             nsrc=4, precision="fp64", method="gmres", restart=30, tol=1e-10),
        # many problems at once: the batch workload's grids, four streams, step graphs
        dict(name="batch-12", kind="batch", count=12, streams=4),
        # the operator by itself on a ragged box
        dict(name="apply-a-ragged", kind="apply_a", nx=200, ny=161, nz=97, bc=DNS, kh=0.3, damp=0.01),
        # the preconditioner by itself, FP64: a ragged box, and the paper's finest grid (h = 1/512)
        dict(name="pinv-ragged", kind="pinv", nx=160, ny=97, nz=200, bc=DNS, kh=0.3, damp=0.01),
        dict(name="pinv-table-511", kind="pinv", nx=511, ny=511, nz=511, bc="DDDDND", kh=20 / 512, damp=0.0),
        # right-hand sides: the dns-256 workload's eight Gaussians, and a separable source
        # of a few terms (what the manufactured problems of the paper's tables hand over)
        dict(name="rhs-gaussians-256", kind="rhs_gaussians", nx=256, ny=256, nz=256, bc=DNS, kh=80 / 257, damp=0.01,
             nsrc=8),
        dict(name="rhs-separable-127", kind="rhs_separable", nx=127, ny=127, nz=127, bc="DDDDSS", kh=20 / 128, damp=0.0,
             nterms=6),
        # the learned correction: one evaluation (what a flexible solve calls per
        # step) and the gradients of one training pair (what a training step computes)
        dict(name="net-forward-128", kind="net_forward", nx=128, ny=128, nz=128, bc=DNS, kh=40 / 129, damp=0.01),
        dict(name="net-gradients-64", kind="net_gradients", nx=64, ny=64, nz=64, bc=DNS, kh=20 / 65, damp=0.01),
    ]


def _axis(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("solve", "solve", "solve", "pinv", "pinv", "apply_a", "rhs_gaussians", "rhs_separable",
                       "batch", "net_forward", "net_gradients"))
    if kind == "batch":
        return dict(kind="batch", count=rng.randint(4, 12), streams=rng.choice((2, 4)))
    if kind in ("net_forward", "net_gradients"):
        hi = 128 if kind == "net_forward" else 64
        nx, ny, nz = (_axis(rng, 20, hi) for _ in range(3))
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, bc=DNS, kh=rng.uniform(0.1, 0.3), damp=0.01)
    hi = dict(pinv=300, solve=200).get(kind, 256)
    nx, ny, nz = (_axis(rng, 24, hi) for _ in range(3))
    if rng.random() < 0.25:                     # a cube: 2^p - 1 (the paper's grids), 2^p or 3 * 2^p interior nodes
        nx = ny = nz = rng.choice((31, 32, 48, 63, 64, 96, 127, 128, 255, 256))
    bc = rng.choice((DNS, DNS, "DDDDDD", "DDDDND", "DDDDSS", "NNNNSS"))
    kh = rng.uniform(0.06, 0.3)
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, bc=bc, kh=kh, damp=0.01)
    if kind == "solve":
        c["bc"] = bc = DNS if bc == "NNNNSS" else bc
        c["precision"] = rng.choice(("fp64", "mixed"))
        # the stationary iteration on the absorbing faces it is used with, GMRES on all of them
        if bc == DNS and rng.random() < 0.5:
            c["method"] = "sks"
        else:
            c["method"] = "gmres" if c["precision"] == "fp64" else "fgmres"
        if nx * ny * nz > 150 ** 3:
            c["kh"] = min(kh, 0.2)
        # at 1e-11 the solution no longer shows the complex64 preconditioner's rounding
        c.update(nsrc=rng.randint(1, 8), restart=rng.choice((20, 30)),
                 tol=1e-10 if c["precision"] == "fp64" else 1e-11)
    elif kind == "rhs_gaussians":
        c["nsrc"] = rng.randint(1, 16)
    elif kind == "rhs_separable":
        c["nterms"] = rng.randint(1, 8)
    return c


# ------------------------------------------------------------------ inputs

def _grid(c):
    n = (c["nx"], c["ny"], c["nz"])
    h = 1.0 / (max(n) + 1)
    k = (c["kh"] / h) * (1 + 1j * c["damp"])
    return n, h, k


def _dims(c):
    bc = c["bc"]
    return tuple(n + (bc[2 * a] != "D") + (bc[2 * a + 1] != "D") for a, n in enumerate((c["nx"], c["ny"], c["nz"])))


def _nodes(c, a):
    """Coordinates of the unknowns on axis a."""
    n, h, _ = _grid(c)
    lo = 1 if c["bc"][2 * a] == "D" else 0
    return (lo + np.arange(_dims(c)[a])) * h


def _sources(c, seed):
    """Seeded Gaussian sources in the middle half of the box, width 4h."""
    n, h, _ = _grid(c)
    rng = np.random.default_rng(seed)
    length = (np.array(n) + 1) * h
    centres = rng.uniform(0.25, 0.75, size=(c["nsrc"], 3)) * length
    amps = rng.standard_normal(c["nsrc"]) + 1j * rng.standard_normal(c["nsrc"])
    return centres, amps, 4.0 * h


def _factors(c, seed):
    """A separable source of a few terms: products of sines of a phase (with
    their derivatives up to order 4), as manufactured solutions give."""
    rng = np.random.default_rng(seed)
    nt = c["nterms"]
    coef = rng.standard_normal(nt) + 1j * rng.standard_normal(nt)
    tabs = []
    for a in range(3):
        w, ph = rng.uniform(1.0, 8.0, nt) * np.pi, rng.uniform(0.0, np.pi, nt)
        x = _nodes(c, a)
        tabs.append(np.stack([np.stack([w[s] ** o * np.sin(w[s] * x + ph[s] + o * np.pi / 2) for o in range(5)])
                              for s in range(nt)]).astype(np.complex128))
    return coef, tabs


def _field(shape, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    return torch.randn(shape, dtype=torch.complex128, device="cuda", generator=g)


def _smooth_field(c, seed):
    """A residual-like field: Gaussians on top of a little noise."""
    coef, tabs = _gauss_tables(dict(c, nsrc=4), seed)
    f = _outer(coef, tabs)
    return f + 0.01 * _field(f.shape, seed + 1)


def _plan(c):
    n, h, k = _grid(c)
    return h6.Plan(n, h, k, c["bc"], precision=c.get("precision", "fp64"))


def _batch_problems(c, seed):
    rng = np.random.default_rng(seed)
    out = []
    sizes = (48, 64, 96, 128, 160)
    for i in range(c["count"]):
        # the sizes in turn (every seed is the same amount of work), wavenumber, faces and source drawn
        n = sizes[i % len(sizes)]
        out.append(dict(nx=n, ny=n, nz=n, bc="DDDDDD" if i % 2 else DNS, kh=float(rng.uniform(10.0, 30.0)) / (n + 1),
                        damp=0.01, nsrc=1, precision="mixed", seed=int(rng.integers(1 << 30))))
    return out


def prepare(c, seed):
    kind = c["kind"]
    if kind == "solve":
        plan = _plan(c)
        F = plan.rhs_gaussians(*_sources(c, seed))
        return dict(kind=kind, case=c, plan=plan, F=F, U=torch.empty_like(F))
    if kind == "batch":
        plans, Fs = [], []
        for p in _batch_problems(c, seed):
            plan = _plan(p)
            plans.append(plan)
            Fs.append(plan.rhs_gaussians(*_sources(p, p["seed"])))
            plan.set_graphs(True)
        return dict(kind=kind, case=c, plans=plans, Fs=Fs, Us=[torch.zeros_like(F) for F in Fs])
    if kind in ("apply_a", "pinv"):
        plan = _plan(c)
        x = _field(plan.shape, seed)
        return dict(kind=kind, plan=plan, x=x, out=torch.empty_like(x))
    if kind == "rhs_gaussians":
        plan = _plan(c)
        return dict(kind=kind, plan=plan, args=_sources(c, seed), out=plan.empty())
    if kind == "rhs_separable":
        plan = _plan(c)
        coef, tabs = _factors(c, seed)
        return dict(kind=kind, plan=plan, args=(coef, *tabs), out=plan.empty())
    if kind in ("net_forward", "net_gradients"):
        plan = _plan(c)
        net = h6.Net(plan.dims)
        net.set_params(_net_params(seed))
        s = dict(kind=kind, plan=plan, net=net, kh=c["kh"], r=_smooth_field(c, seed))
        if kind == "net_forward":
            s["out"] = torch.empty_like(s["r"])
        else:
            s["t"] = 0.05 * _smooth_field(c, seed + 100)
        return s
    raise ValueError(kind)


def _net_params(seed):
    p = init_net_params(h6.NET_LAYERS, seed)
    w, b = p["out"]
    p["out"] = (30.0 * w, b)           # a correction of the size a trained network gives
    return h6.pack_net_params(p)


def run(s):
    kind = s["kind"]
    if kind == "solve":
        c = s["case"]
        U, info = s["plan"].solve(s["F"], s["U"], method=c["method"], restart=c["restart"], tol=c["tol"], maxit=500,
                                  zero_guess=True)
        # (in a mixed plan the step at which the tolerance is met depends on complex64 rounding)
        return {"U": U, "iters": info["iters"]} if c["precision"] == "fp64" else {"U": U}
    if kind == "batch":
        for U in s["Us"]:
            U.zero_()
        h6.solve_batch(s["plans"], s["Fs"], s["Us"], method="fgmres", restart=30, tol=1e-11, maxit=600,
                       nstreams=s["case"]["streams"])
        return {"U": s["Us"]}
    if kind == "apply_a":
        return s["plan"].apply_A(s["x"], s["out"])
    if kind == "pinv":
        return s["plan"].apply_Pinv(s["x"], s["out"])
    if kind == "rhs_gaussians":
        return s["plan"].rhs_gaussians(*s["args"], out=s["out"])
    if kind == "rhs_separable":
        return s["plan"].rhs_separable(*s["args"], out=s["out"])
    if kind == "net_forward":
        return s["net"].forward(s["r"], s["kh"], s["out"])
    loss, grads = s["net"].gradients_op(s["plan"], s["r"], s["t"])
    return {"loss": loss, "grads": grads}


# ------------------------------------------------------------------ least work

def _pinv_flops(c):
    """Fast transforms (5 L log2 L per complex line of length L, both ways) and a tridiagonal solve."""
    nx, ny, nz = _dims(c)
    return nx * ny * nz * (10.0 * (math.log2(nx + 2) + math.log2(ny + 2)) + 30.0)


def _net_flops(dims):
    g1 = list(dims)
    g2 = [(x + 1) // 2 for x in g1]
    g3 = [(x + 1) // 2 for x in g2]
    size = [float(np.prod(g)) for g in (g1, g2, g3)]
    level = dict(e1a=0, e1b=0, e2a=1, e2b=1, b3a=2, b3b=2, d2a=1, d2b=1, d1a=0, d1b=0, out=0)
    return sum(2.0 * 27 * ci * co * size[level[name]] for name, ci, co in h6.NET_LAYERS)


def work(c):
    kind = c["kind"]
    if kind == "batch":
        parts = [work(dict(p, kind="solve")) for p in _batch_problems(c, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    N = float(np.prod(_dims(c)))
    if kind == "solve":
        # a nominal number of steps, each one operator and one preconditioner application
        steps = 4 + 30 * c["kh"]
        return {"bytes": N * (32 + 64 * steps), "flops": steps * (N * 110 + _pinv_flops(c))}
    if kind == "apply_a":
        return {"bytes": 32 * N, "flops": 110 * N}
    if kind == "pinv":
        return {"bytes": 32 * N, "flops": _pinv_flops(c)}
    if kind == "rhs_gaussians":
        return {"bytes": 16 * N, "flops": 12.0 * c["nsrc"] * N}
    if kind == "rhs_separable":
        return {"bytes": 16 * N, "flops": 24.0 * c["nterms"] * N}
    f = _net_flops(_dims(c))
    if kind == "net_forward":
        return {"bytes": 32 * N, "flops": f}
    return {"bytes": 32 * N, "flops": 3 * f}


# ------------------------------------------------------------------ the same in 64 bits, plain torch

def _second_diff(U, dim, lo, hi):
    """h^2 times the 3-point second difference; ghosts 0 next to a Dirichlet
    face, the mirror value next to a Neumann one."""
    V = U.movedim(dim, 0)
    out = -2.0 * V
    out[1:] += V[:-1]
    out[:-1] += V[1:]
    if V.shape[0] > 1:
        if lo == "N":
            out[0] += V[1]
        if hi == "N":
            out[-1] += V[-2]
    return out.movedim(0, dim)


def _exact_a(c, U):
    """The h^2-scaled sixth-order compact operator D_z G + P with its closure rows."""
    _, h, k = _grid(c)
    bc, kap, ikh = c["bc"], (k * h) ** 2, 1j * k * h
    a = (1 + kap / 30) / 6

    def plane(V, c_id, c_lap, c_mix):
        dx = _second_diff(V, -1, bc[0], bc[1])
        return c_id * V + c_lap * (dx + _second_diff(V, -2, bc[2], bc[3])) + c_mix * _second_diff(dx, -2, bc[2], bc[3])

    G = plane(U, 1.0, a, 1 / 30)
    out = plane(U, kap * (1 - kap / 12 + kap ** 2 / 360), 1.0, a) - 2.0 * G
    out[1:] += G[:-1]
    out[:-1] += G[1:]
    mu3 = 1 / (1 + (2 * ikh / 3) * (1 + 2 * kap / 15))
    mu1 = (ikh / 90 + (1 + kap / 30) / (6 * mu3)) / (1 + 2 * ikh / 3)
    q, r = np.exp(2 * ikh) * mu3, np.exp(ikh) * mu3
    kh3 = (k * h) ** 3
    for face, edge, inner in ((bc[4], 0, 1), (bc[5], -1, -2)):
        if U.shape[0] < 2 or face == "D":
            continue
        if face == "N":
            out[edge] += G[inner]
        else:
            out[edge] += plane(U[inner], q * (1 - 2 * ikh / 3 - 4j * kh3 / 45),
                               q * (mu1 + (2 * ikh / 3) * (1 / 60 - mu1)), q / (30 * mu3))
            out[edge] += plane(U[edge], r * (4 * ikh / 3) * (1 + 2 * kap / 15), -r * (4 * ikh / 3) * (1 / 60 - mu1), 0.0)
    return out


class _ExactPinv:
    """The inverse of the 7-point operator: basis products along x and y, Thomas along z."""

    def __init__(self, c):
        _, h, k = _grid(c)
        self.bc, self.dims = c["bc"], _dims(c)
        kap = (k * h) ** 2
        self.mats, lam = [], []
        for a in range(2):
            L, M = self.dims[a], (c["nx"], c["ny"])[a] + 1
            if self.bc[2 * a] == "D":
                i = torch.arange(1, L + 1, dtype=torch.int64, device="cuda")
                B = torch.sin(math.pi / M * ((i[:, None] * i[None, :]) % (2 * M)).double())
                F = (2.0 / M) * B
            else:
                i = torch.arange(L, dtype=torch.int64, device="cuda")
                B = torch.cos(math.pi / M * ((i[:, None] * i[None, :]) % (2 * M)).double())
                w = torch.ones(L, dtype=torch.float64, device="cuda")
                w[0] = w[-1] = 0.5
                F = (2.0 / M) * w[:, None] * B * w[None, :]
            self.mats.append((F, B))
            lam.append(-4.0 * torch.sin(math.pi / (2 * M) * i.double()) ** 2)
        self.shift = kap + lam[0][None, :] + lam[1][:, None].to(torch.complex128)
        nz = self.dims[2]
        self.end = 2j * k * h
        self.lo, self.hi = self.bc[4], self.bc[5]
        self.nz = nz
        self.cp, self.piv = [], []
        for l in range(nz):
            d = self.shift - 2.0 + self.end * ((l == 0 and self.lo == "S") + (l == nz - 1 and self.hi == "S"))
            if l > 0:
                d = d - self._sub(l) * self.cp[l - 1]
            self.piv.append(d)
            self.cp.append(self._sup(l) / d)

    def _sub(self, l):
        return 2.0 if l == self.nz - 1 and self.hi != "D" and self.nz > 1 else 1.0

    def _sup(self, l):
        return 2.0 if l == 0 and self.lo != "D" and self.nz > 1 else 1.0

    def _x(self, V, W):
        R = torch.view_as_real(V).movedim(-1, 0).reshape(-1, V.shape[-1])
        R = (R @ W.T).reshape(2, *V.shape)
        return torch.complex(R[0], R[1])

    def _y(self, V, W):
        return self._x(V.transpose(1, 2).contiguous(), W).transpose(1, 2).contiguous()

    def __call__(self, R):
        V = self._y(self._x(R, self.mats[0][0]), self.mats[1][0])
        for l in range(self.nz):
            V[l] = (V[l] - self._sub(l) * V[l - 1]) / self.piv[l] if l > 0 else V[0] / self.piv[0]
        for l in range(self.nz - 2, -1, -1):
            V[l] -= self.cp[l] * V[l + 1]
        return self._x(self._y(V, self.mats[1][1]), self.mats[0][1])


def _exact_solve(c, F, tol=3e-12, m=40, most=200):
    """Right-preconditioned GMRES(m) to a residual far below the cases'
    tolerances (or until rounding stops its fall)."""
    P, N = _ExactPinv(c), F.numel()
    U, normF, done, last = torch.zeros_like(F), float(torch.linalg.norm(F)), 0, math.inf
    while done < most:
        r = F - _exact_a(c, U)
        beta = float(torch.linalg.norm(r))
        if beta <= tol * normF or beta > 0.3 * last:
            break
        last = beta
        V = torch.empty((m + 1, N), dtype=torch.complex128, device="cuda")
        V[0] = r.reshape(-1) / beta
        H = np.zeros((m + 1, m), dtype=np.complex128)
        y = None
        for j in range(m):
            w = _exact_a(c, P(V[j].reshape(F.shape))).reshape(-1)
            for _ in range(2):                      # Gram-Schmidt, twice
                for i in range(j + 1):
                    s = torch.vdot(V[i], w)
                    H[i, j] += complex(s)
                    w -= s * V[i]
            H[j + 1, j] = float(torch.linalg.norm(w))
            V[j + 1] = w / H[j + 1, j].real
            e = np.zeros(j + 2, dtype=np.complex128)
            e[0] = beta
            y, res = np.linalg.lstsq(H[:j + 2, :j + 1], e, rcond=None)[:2]
            done += 1
            if np.linalg.norm(H[:j + 2, :j + 1] @ y - e) <= 0.3 * tol * normF:
                break
        w = torch.zeros_like(V[0])
        for i, s in enumerate(y):
            w += complex(s) * V[i]
        U = U + P(w.reshape(F.shape))
    return U


def _gauss_tables(c, seed):
    centres, amps, sigma = _sources(c, seed)
    tabs = []
    for a in range(3):
        t = (_nodes(c, a)[None, :] - centres[:, a:a + 1]) / sigma
        he = (np.ones_like(t), t, t ** 2 - 1, t ** 3 - 3 * t, t ** 4 - 6 * t ** 2 + 3)
        tabs.append(np.stack([(-1 / sigma) ** o * he[o] * np.exp(-0.5 * t ** 2) for o in range(5)], 1).astype(np.complex128))
    return amps, tabs


def _outer(coef, tabs, orders=(0, 0, 0)):
    """sum_s coef_s X_s(x) Y_s(y) Z_s(z) of the factors' derivatives of the given orders."""
    x, y, z = (torch.from_numpy(np.ascontiguousarray(t[:, o])).cuda() for t, o in zip(tabs, orders))
    cz = torch.from_numpy(np.asarray(coef, dtype=np.complex128)).cuda()[:, None] * z
    yz = (cz[:, :, None] * y[:, None, :]).reshape(len(coef), -1)
    return (yz.T.contiguous() @ x).reshape(z.shape[1], y.shape[1], x.shape[1])


def _exact_rhs(c, coef, tabs):
    """h^2 times the compact right-hand side with its face terms."""
    n, h, k = _grid(c)
    bc, kap, ikh = c["bc"], (k * h) ** 2, 1j * k * h

    def d(ox, oy, oz, sel=None):
        t = list(tabs)
        if sel is not None:                         # one plane only: (axis, index)
            t[sel[0]] = t[sel[0]][:, :, sel[1]:sel[1] + 1]
        return _outer(coef, t, (ox, oy, oz))

    def lap(sel=None):
        return d(2, 0, 0, sel) + d(0, 2, 0, sel) + d(0, 0, 2, sel)

    mix = d(2, 2, 0) + d(2, 0, 2) + d(0, 2, 2)
    F = h ** 2 * ((1 - kap / 12 + kap ** 2 / 360) * d(0, 0, 0) + (h ** 2 / 12) * (1 - kap / 30) * lap()
                  + (h ** 4 / 360) * (d(4, 0, 0) + d(0, 4, 0) + d(0, 0, 4) + 2 * mix) + (h ** 4 / 180) * mix)
    view = {0: lambda i: F[:, :, i:i + 1], 1: lambda i: F[:, i:i + 1, :], 2: lambda i: F[i:i + 1]}
    e = np.eye(3, dtype=int)
    mu3 = 1 / (1 + (2 * ikh / 3) * (1 + 2 * kap / 15))
    mu1 = (ikh / 90 + (1 + kap / 30) / (6 * mu3)) / (1 + 2 * ikh / 3)
    for a in range(3):
        for side in range(2):
            i = 0 if side == 0 else _dims(c)[a] - 1
            face, sel, sg = bc[2 * a + side], (a, i), 1.0 if side == 0 else -1.0
            if face == "N":
                t1, t2 = [b for b in range(3) if b != a]
                RN = ((h ** 2 / 6) * (1 - kap / 20) * d(*e[a], sel) + (h ** 4 / 120) * d(*(3 * e[a]), sel)
                      + (7 * h ** 4 / 360) * (d(*(e[a] + 2 * e[t1]), sel) + d(*(e[a] + 2 * e[t2]), sel)))
                view[a](i).add_(sg * 2 * h * RN)
            elif face == "S":
                ik = 1j * k
                f0, f1, f2, f3 = d(0, 0, 0, sel), sg * d(0, 0, 1, sel), d(0, 0, 2, sel), sg * d(0, 0, 3, sel)
                b1 = ik * f0 + f1
                b2 = ik ** 2 * f0 + 2 * ik * f1 + f2
                b3 = ik ** 3 * f0 + 3 * ik ** 2 * f1 + 3 * ik * f2 + f3
                Lb = ik * (d(2, 0, 0, sel) + d(0, 2, 0, sel)) + sg * (d(2, 0, 1, sel) + d(0, 2, 1, sel))
                Fb = (h ** 2 / 6 + k ** 2 * h ** 4 / 45) * b1 - (ik * h ** 4 / 90) * b2 + (h ** 4 / 120) * (b3 - Lb)
                view[a](i).add_(np.exp(ikh) * mu3 * (2 * h * Fb + mu1 * (h ** 5 / 3) * Lb))
    return F


def _conv(x, w, b):
    """3 x 3 x 3 convolution, zero outside; x: (Z, Y, X, Cin), w: (Cout, Cin, 3, 3, 3)."""
    Z, Y, X, ci = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    out = b.repeat(Z * Y * X, 1)
    for dz in range(3):
        for dy in range(3):
            for dx in range(3):
                out = out + p[dz:dz + Z, dy:dy + Y, dx:dx + X].reshape(-1, ci) @ w[:, :, dz, dy, dx].T
    return out.reshape(Z, Y, X, -1)


def _pool(x):
    Z, Y, X, c = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 0, X % 2, 0, Y % 2, 0, Z % 2))
    return p.reshape((Z + 1) // 2, 2, (Y + 1) // 2, 2, (X + 1) // 2, 2, c).sum((1, 3, 5)) / 8


def _up(x, like):
    Z, Y, X = like.shape[:3]
    return x.repeat_interleave(2, 0)[:Z].repeat_interleave(2, 1)[:, :Y].repeat_interleave(2, 2)[:, :, :X]


def _exact_net(c, seed, r, params=None):
    """(scale s, output y (P, 2)) of the network on the residual r in 64 bits."""
    if params is None:
        params = {n: (torch.from_numpy(np.array(w, dtype=np.float64)).cuda(), torch.from_numpy(np.array(b, dtype=np.float64)).cuda())
                  for n, (w, b) in h6.unpack_net_params(_net_params(seed)).items()}
    s = torch.sqrt((r.abs() ** 2).mean())
    x = torch.stack([r.real / s, r.imag / s, torch.full_like(r.real, c["kh"])], -1)

    def layer(name, v):
        return torch.relu(_conv(v, *params[name]))

    s1 = layer("e1b", layer("e1a", x))
    s2 = layer("e2b", layer("e2a", _pool(s1)))
    b3 = layer("b3b", layer("b3a", _pool(s2)))
    d2 = layer("d2b", layer("d2a", torch.cat([_up(b3, s2), s2], -1)))
    d1 = layer("d1b", layer("d1a", torch.cat([_up(d2, s1), s1], -1)))
    return s, _conv(d1, *params["out"]), params


def exact(c, seed):
    kind = c["kind"]
    if kind == "solve":
        F = _exact_rhs(c, *_gauss_tables(c, seed))
        U = _exact_solve(c, F)
        return {"U": U, "iters": None} if c["precision"] == "fp64" else {"U": U}
    if kind == "batch":
        ps = _batch_problems(c, seed)
        return {"U": [_exact_solve(p, _exact_rhs(p, *_gauss_tables(p, p["seed"]))) for p in ps]}
    if kind == "apply_a":
        return _exact_a(c, _field(_dims(c)[::-1], seed))
    if kind == "pinv":
        return _ExactPinv(c)(_field(_dims(c)[::-1], seed))
    if kind == "rhs_gaussians":
        return _exact_rhs(c, *_gauss_tables(c, seed))
    if kind == "rhs_separable":
        return _exact_rhs(c, *_factors(c, seed))
    r = _smooth_field(c, seed)
    if kind == "net_forward":
        with torch.no_grad():
            s, y, _ = _exact_net(c, seed, r)
        return s * torch.complex(y[..., 0], y[..., 1])
    params = {n: (torch.from_numpy(np.array(w, dtype=np.float64)).cuda().requires_grad_(),
                  torch.from_numpy(np.array(b, dtype=np.float64)).cuda().requires_grad_())
              for n, (w, b) in h6.unpack_net_params(_net_params(seed)).items()}
    s, y, _ = _exact_net(c, seed, r, params)
    with torch.no_grad():
        t = 0.05 * _smooth_field(c, seed + 100)
        u = _exact_a(c, s * torch.complex(y[..., 0], y[..., 1]) - t)
        den = float((_exact_a(c, t).abs() ** 2).sum())
        g = (2.0 / den) * s * _exact_a(c, u.conj().resolve_conj()).conj()
        dy = torch.stack([g.real, g.imag], -1)
    y.backward(dy)
    grads = torch.cat([p.grad.reshape(-1) for name, _, _ in h6.NET_LAYERS for p in params[name]])
    return {"loss": float((u.abs() ** 2).sum()) / den, "grads": grads.cpu().numpy()}
