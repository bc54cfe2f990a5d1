"""Workloads of the space-time heat solver: what a program that uses it calls.

A case is one call through the public entry points of `paper_1802_09277_amd`:
a solve to the working tolerance 1e-8 from a zero guess (V-cycles in either
iteration basis, or FGMRES), or one of the operators that a program with an
outer iteration of its own calls (V-cycle, smoother, slab inverse, residual).
The shapes are those of the repository's benchmark configurations and of its
serving mix, and generic ones between them: unit square or cube, spline
degrees 1 to 4, from 16 thousand to 201 million unknowns.
"""
import math

import numpy as np
import torch

import paper_1802_09277_amd as sth

RTOL = 1e-8                     # the tolerance of every solve
THETA, OMEGA = 0.01, 0.5        # the solver's defaults (final time 1)
MODES = 8                       # separable modes of a right-hand side


def _case(name, call, dim, n_elem, degree, n_slabs, n_elem_t, **more):
    c = {"name": name, "call": call, "dim": dim, "n_elem": n_elem, "degree": degree, "n_slabs": n_slabs,
         "n_elem_t": n_elem_t, "basis": "nodal", "prec": "fp64", "coarse_slabs": 128, "space_ratio": 0.0}
    c.update(more)
    return c


def listed():
    return [
        # the smallest benchmark configuration: one exact level, a call that
        # is all launches and latency (a time step of a parameter study)
        _case("solve_small", "solve", 2, 16, 2, 16, 2, basis="eigen"),
        # the middle benchmark configuration: cubic splines, 256 slabs, the
        # typical size of a served request
        _case("solve_mid", "solve", 2, 64, 3, 256, 2, basis="eigen"),
        # the largest benchmark configuration, 201 million unknowns: a
        # production run that fills the card
        _case("solve_large", "solve", 2, 256, 2, 1024, 1, basis="eigen"),
        # the mixed-precision form (FP32 transforms and eigenbasis vectors,
        # FP64 defect correction) on the same mesh, a quarter of the slabs
        _case("solve_mixed", "solve", 2, 256, 2, 256, 1, basis="eigen", prec="fp32"),
        # the heaviest kind of request of the serving mix: quartic splines on
        # the finest mesh, 258 functions per axis
        _case("solve_quartic", "solve", 2, 256, 4, 64, 2, basis="eigen"),
        # the 3-D benchmark configuration with two levels in time
        _case("solve_cube", "solve", 3, 32, 2, 128, 2, basis="eigen", coarse_slabs=64),
        # the binding's default iteration (B-spline coefficients) on a mesh
        # and slab count that are no powers of two
        _case("solve_nodal", "solve", 2, 60, 3, 192, 2, coarse_slabs=48),
        # the multigrid as a preconditioner of flexible GMRES, also in the
        # default basis, linear splines
        _case("fgmres", "fgmres", 2, 80, 1, 160, 2, coarse_slabs=40),
        # one V-cycle inside a program's own outer iteration, odd sizes
        _case("vcycle", "vcycle", 2, 101, 2, 300, 1),
        # two smoothing steps on a cubic 3-D mesh (22 functions per axis):
        # the smoother as a component of another multigrid
        _case("smooth", "smooth", 3, 21, 3, 50, 1),
        # the slab inverse of a few slabs: the block-Jacobi preconditioner,
        # small enough for launches to count
        _case("slab_inverse", "block_solve", 2, 40, 2, 24, 2),
        # the residual of a 3-D space-time vector, a matrix-free operator
        # that Krylov methods and error estimators call
        _case("residual", "residual", 3, 33, 2, 100, 2),
    ]


def _unknowns(c):
    return c["n_slabs"] * (c["n_elem_t"] + c["degree"]) * (c["n_elem"] + c["degree"] - 2) ** c["dim"]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        call = rng.choice(["solve", "solve", "solve", "solve", "fgmres", "vcycle", "smooth", "block_solve", "residual"])
        dim = rng.choice([2, 2, 2, 3])
        c = _case("", call, dim, log(12, 256) if dim == 2 else log(6, 40), rng.choice([1, 2, 2, 3, 3, 4]), log(8, 1024),
                  rng.choice([1, 2, 2]))
        del c["name"]
        if rng.random() < 0.5:          # slab counts that can be halved several times, as the multigrid likes them
            c["n_slabs"] = max(8, c["n_slabs"] // 8 * 8)
        if call in ("solve", "fgmres", "vcycle") and rng.random() < 0.5:
            c["coarse_slabs"] = max(4, c["n_slabs"] // rng.choice([2, 4, 8]))
        if call in ("solve", "fgmres"):
            c["basis"] = rng.choice(["eigen", "eigen", "nodal"])
        if call == "solve" and c["basis"] == "nodal" and rng.random() < 0.3:
            c["space_ratio"] = 2.0
        if call == "solve" and c["basis"] == "eigen" and rng.random() < 0.2:
            c["prec"] = rng.choice(["fp32", "bf16x3"])
        most = 3e7 if call in ("solve", "fgmres") else 6e7
        if c["basis"] == "nodal" and call in ("solve", "fgmres"):
            most = 8e6
        if 1e4 <= _unknowns(c) <= most:
            return c


class _Modes:
    """f = sum_m amp prod_a sin(k_a pi x_a) cos(omega pi t): wave numbers 1
    to 8, frequencies 0 to 4, normal amplitudes."""

    def __init__(self, seed, dim):
        rng = np.random.default_rng(seed)
        self.amp = rng.standard_normal(MODES)
        self.k = rng.integers(1, 9, size=(MODES, dim))
        self.omega = rng.integers(0, 5, size=MODES).astype(np.float64)

    def arrays(self):
        return self.amp, self.k, self.omega, np.zeros(MODES)


def _normal(seed, stream, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 16 + stream)
    return torch.randn(n, generator=g, dtype=torch.float64, device="cuda")


def _iterate(case, seed, n):
    """An iterate with every frequency in it, of the size of the solutions."""
    return _normal(seed, 1, n).mul_(1e-3)


def prepare(case, seed):
    solver = sth.Solver(case["dim"], case["n_elem"], case["degree"], case["n_slabs"], case["n_elem_t"], theta=THETA,
                        omega=OMEGA, prec=case["prec"], coarse_slabs=case["coarse_slabs"], basis=case["basis"],
                        space_ratio=case["space_ratio"])
    state = {"call": case["call"], "solver": solver}
    if case["call"] == "block_solve":
        state["f"] = _normal(seed, 0, solver.vector_len)
        state["u"] = solver.new_vector()
        return state
    state["f"] = solver.load_rhs(_Modes(seed, case["dim"]), solver.new_vector())
    if case["call"] in ("solve", "fgmres"):
        state["u"] = solver.new_vector()
    else:
        state["u"] = _iterate(case, seed, solver.vector_len)
    if case["call"] == "residual":
        state["r"] = solver.new_vector()
    return state


def run(state):
    s, f, u = state["solver"], state["f"], state["u"]
    call = state["call"]
    if call == "solve":
        iters, _, _ = s.solve(f, u.zero_(), rtol=RTOL, maxit=100)
        return {"u": u, "iters": iters}
    if call == "fgmres":
        iters, _, _ = s.solve_fgmres(f, u.zero_(), rtol=RTOL, maxit=100, restart=20)
        return {"u": u, "iters": iters}
    if call == "vcycle":
        return {"u": s.vcycle(f, u)}
    if call == "smooth":
        return {"u": s.smooth(f, u, steps=2)}
    if call == "block_solve":
        return {"z": s.block_solve(f, u)}
    return {"r": s.residual(f, u, state["r"])}


def work(case):
    """Vectors read and written once; multiply-adds of the transforms into
    and out of the spatial eigenbasis (they are what a slab inverse takes),
    or of the banded stencils for the residual."""
    dof, n, dim = _unknowns(case), case["n_elem"] + case["degree"] - 2, case["dim"]
    nt, band = case["n_elem_t"] + case["degree"], 2 * case["degree"] + 1
    if case["call"] == "residual":
        return {"bytes": 24.0 * dof, "flops": dof * (2.0 * (2 * dim) * band + 4.0 * nt + 2.0)}
    vectors = 2.0 if case["call"] in ("solve", "fgmres", "block_solve") else 3.0
    return {"bytes": 8.0 * vectors * dof, "flops": 2.0 * dof * dim * 2.0 * n}


# ---------------------------------------------------------------------------
# The same results in 64-bit torch and numpy: 1-D Galerkin matrices by Gauss
# quadrature, generalised eigenvectors of the spatial pencil, and per spatial
# mode the small temporal systems.
# ---------------------------------------------------------------------------
def _basis(knots, p, xs):
    """Values and first derivatives of every B-spline at xs (points x functions)."""
    xs = np.asarray(xs, dtype=np.float64)
    nk = len(knots) - 1
    last = max(i for i in range(nk) if knots[i] < knots[i + 1])
    v = np.zeros((len(xs), nk))
    for i in range(nk):
        if knots[i] < knots[i + 1]:
            v[:, i] = (xs >= knots[i]) & ((xs < knots[i + 1]) | ((i == last) & (xs <= knots[i + 1])))
    d = np.zeros_like(v)
    for q in range(1, p + 1):
        w, dw = np.zeros((len(xs), nk - q)), np.zeros((len(xs), nk - q))
        for i in range(nk - q):
            left, right = knots[i + q] - knots[i], knots[i + q + 1] - knots[i + 1]
            if left > 0:
                w[:, i] += (xs - knots[i]) / left * v[:, i]
                dw[:, i] += q / left * v[:, i]
            if right > 0:
                w[:, i] += (knots[i + q + 1] - xs) / right * v[:, i + 1]
                dw[:, i] -= q / right * v[:, i + 1]
        v, d = w, dw
    return v, d


def _knots(a, b, n, p):
    return np.concatenate([[a] * p, np.linspace(a, b, n + 1), [b] * p])


def _gauss(a, b, n, q):
    x, w = np.polynomial.legendre.leggauss(q)
    e = np.linspace(a, b, n + 1)
    half = (e[1:] - e[:-1]) / 2
    return (((e[1:] + e[:-1]) / 2)[:, None] + half[:, None] * x).ravel(), (half[:, None] * w).ravel()


class _Exact:
    def __init__(self, case):
        self.c = case
        self.dim, self.p, self.S = case["dim"], case["degree"], case["n_slabs"]
        self.ne, self.net = case["n_elem"], case["n_elem_t"]
        self.n, self.nt = self.ne + self.p - 2, self.net + self.p
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        knots = _knots(0.0, 1.0, self.ne, self.p)
        x, w = _gauss(0.0, 1.0, self.ne, self.p + 1)
        v, d = (a[:, 1:-1] for a in _basis(knots, self.p, x))
        self.M, self.K = (v * w[:, None]).T @ v, (d * w[:, None]).T @ d
        chol = np.linalg.cholesky(self.M)
        inv = np.linalg.inv(chol)
        lam, q = np.linalg.eigh(inv @ self.K @ inv.T)
        self.U = inv.T @ q
        one = lam
        for _ in range(self.dim - 1):
            one = (one[..., None] + lam).reshape(-1)
        self.mu = self._t(one)

    def _t(self, a):
        return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=self.dev)

    def time(self, level):
        """K_t and M_t of a level's slabs (twice as long on each, the finest
        level's upwind parameter)."""
        tau = 1.0 / self.S * 2 ** level
        sigma = THETA / self.S / self.net
        knots = _knots(0.0, tau, self.net, self.p)
        x, w = _gauss(0.0, tau, self.net, self.p + 1)
        v, d = _basis(knots, self.p, x)
        test = (v + sigma * d) * w[:, None]
        k, m = test.T @ d, test.T @ v
        k[0, 0] += 1.0
        return k, m

    def load(self, modes):
        amp, k, omega, _ = modes.arrays()
        tau, sigma = 1.0 / self.S, THETA / self.S / self.net
        x, w = _gauss(0.0, tau, self.net, self.p + 3)
        v, d = _basis(_knots(0.0, tau, self.net, self.p), self.p, x)
        test = (v + sigma * d) * w[:, None]
        xs, ws = _gauss(0.0, 1.0, self.ne, self.p + 3)
        space = _basis(_knots(0.0, 1.0, self.ne, self.p), self.p, xs)[0][:, 1:-1] * ws[:, None]
        f = torch.zeros(self.S * self.nt, self.n ** self.dim, dtype=torch.float64, device=self.dev)
        for m in range(len(amp)):
            tt = np.cos(omega[m] * math.pi * (np.arange(self.S)[:, None] * tau + x[None, :])) @ test
            row = np.ones(1)
            for a in reversed(range(self.dim)):         # x is the fastest index
                row = (row[:, None] * (np.sin(k[m, a] * math.pi * xs) @ space)).reshape(-1)
            f.addmm_(self._t(tt.reshape(-1, 1)), self._t(amp[m] * row.reshape(1, -1)))
        return f.view(self.S, self.nt, -1)

    def axes(self, v, mats):
        """One matrix along each spatial axis (x last) of v (slab, time, space)."""
        shape = v.shape
        v = v.reshape((-1,) + (self.n,) * self.dim)
        for a, mat in enumerate(mats):
            if mat is not None:
                v = torch.matmul(v.movedim(a + 1, -1).contiguous(), self._t(mat.T)).movedim(-1, a + 1)
        return v.reshape(shape)

    def mix(self, mat, v):
        out = torch.zeros((v.shape[0], mat.shape[0]) + v.shape[2:], dtype=v.dtype, device=v.device)
        for i in range(mat.shape[0]):
            for j in range(mat.shape[1]):
                if mat[i, j] != 0.0:
                    out[:, i].add_(v[:, j], alpha=float(mat[i, j]))
        return out

    def residual(self, f, u):
        k, m = self.time(0)
        mass = self.axes(u, [self.M] * self.dim)
        r = f - self.mix(k, mass)
        r[1:, 0] += mass[:-1, -1]
        stiff = torch.zeros_like(u)
        for a in range(self.dim):
            stiff += self.axes(u, [self.K if b == a else self.M for b in range(self.dim)])
        return r - self.mix(m, stiff)

    def forward(self, v):
        return self.axes(v, [self.U.T] * self.dim)

    def backward(self, v):
        return self.axes(v, [self.U] * self.dim)

    # below: in the spatial eigenbasis, v is (slab, time, mode) ---------------
    def inverse(self, level):
        k, m = self.time(level)
        a = self._t(k)[None] + self.mu[:, None, None] * self._t(m)[None]
        return torch.linalg.inv(a.cpu()).to(self.dev)

    def solve_slabs(self, inv, v):
        out = torch.zeros_like(v)
        for i in range(self.nt):
            for j in range(self.nt):
                out[:, i].addcmul_(v[:, j], inv[:, i, j].expand_as(v[:, j]))
        return out

    def operator(self, level, u):
        k, m = self.time(level)
        y = self.mix(k, u) + self.mu * self.mix(m, u)
        y[1:, 0] -= u[:-1, -1]
        return y

    def substitute(self, level, f):
        inv = self.inverse(level)
        u = self.solve_slabs(inv, f)
        first = inv[:, :, 0].T.contiguous()             # A^{-1} e_1
        for s in range(1, u.shape[0]):
            u[s] += first * u[s - 1, -1]
        return u

    def prolongation(self, level):
        """Coefficients on two slabs of the functions of one twice as long."""
        tau = 1.0 / self.S * 2 ** level
        x = np.linspace(0.0, tau, 8 * self.nt + 1)
        x = (x[1:] + x[:-1]) / 2
        fine = _basis(_knots(0.0, tau, self.net, self.p), self.p, x)[0]
        coarse = _knots(0.0, 2 * tau, self.net, self.p)
        return np.concatenate([np.linalg.lstsq(fine, _basis(coarse, self.p, x + o)[0], rcond=None)[0] for o in (0.0, tau)])

    def cycle(self, level, f):
        """V(1,1) from zero."""
        slabs = f.shape[0]
        if slabs <= self.c["coarse_slabs"] or slabs % 2:
            return self.substitute(level, f)
        inv, pt = self.inverse(level), self.prolongation(level)
        u = OMEGA * self.solve_slabs(inv, f)
        r = f - self.operator(level, u)
        ec = self.cycle(level + 1, self.mix(pt.T, r.reshape(slabs // 2, 2 * self.nt, -1)))
        u += self.mix(pt, ec).reshape(u.shape)
        return u + OMEGA * self.solve_slabs(inv, f - self.operator(level, u))


def exact(case, seed):
    x = _Exact(case)
    shape = (x.S, x.nt, x.n ** x.dim)
    call = case["call"]
    if call == "block_solve":
        r = _normal(seed, 0, _unknowns(case)).view(shape)
        return {"z": x.backward(x.solve_slabs(x.inverse(0), x.forward(r))).reshape(-1)}
    f = x.load(_Modes(seed, case["dim"]))
    if call in ("solve", "fgmres"):
        return {"u": x.backward(x.substitute(0, x.forward(f))).reshape(-1), "iters": None}
    u = _iterate(case, seed, _unknowns(case)).view(shape)
    if call == "residual":
        return {"r": x.residual(f, u).reshape(-1)}
    if call == "vcycle":
        return {"u": (u + x.backward(x.cycle(0, x.forward(x.residual(f, u))))).reshape(-1)}
    for _ in range(2):
        u = u + OMEGA * x.backward(x.solve_slabs(x.inverse(0), x.forward(x.residual(f, u))))
    return {"u": u.reshape(-1)}
