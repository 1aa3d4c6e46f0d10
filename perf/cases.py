"""Performance cases of the stochastic Galerkin solver.

Each case is one call that a program makes through the Python binding: the SG
operator, a batch of inner solves, one preconditioner action, whole solves with
each preconditioner and inner precision, the quantity-of-interest gradient, the
multi-problem batch and the lognormal solve. ``prepare`` builds the problem, the
handle and the seeded right-hand side on the GPU, ``run`` makes the call,
``exact`` gives the same result in 64 bits from plain torch and numpy, and
``draw`` gives more cases of the same ranges.

Coefficients are the exponential-covariance KL fields of ``sg_inputs``; a case
keeps its coefficient for every seed, and the seed moves the right-hand side,
as in a program that solves for many loads on one model.
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

from sg_inputs import batch_problems, n_chaos, qoi_weights
from sg_inputs.problems import make_problem, nodal_rhs

# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------


def _case(name, op, **kw):
    c = {"name": name, "op": op, "n_e": 16, "M": 4, "p": 2, "sigma": 0.2, "L": 0.5, "family": "hermite"}
    c.update(kw)
    return c


def listed():
    return [
        # the operator on the smallest named problem: a call that is all latency (an outer
        # Krylov method of the caller's own on a coarse model)
        _case("matvec_16", "matvec"),
        # the operator at the benchmark's size, 18.6M unknowns
        _case("matvec_256", "matvec", n_e=256, M=10, p=3, sigma=0.25, L=0.3),
        # an odd grid, uniform variables and a higher degree with fewer terms
        _case("matvec_201_legendre", "matvec", n_e=201, M=6, p=4, sigma=0.2, L=0.5, family="legendre"),
        # a batch of diagonal-block solves on an odd grid, as a caller's own level loop issues it
        _case("inner_101", "inner", n_e=101, M=6, p=2, ncols=28, degree=8, inner_rtol=1e-4),
        # one preconditioner action with the binding's default options on a middle-sized problem
        _case("hsc_action_128", "hsc", n_e=128, M=8, p=3, degree=4, inner_rtol=1e-4),
        # the smallest named solve, inner solves nearly exact as the reference comparison runs it
        _case("solve_16", "solve", degree=4, inner_rtol=1e-12, precision=64, precond="hsc", warm=False, rtol=1e-8),
        # the benchmark's solve, FP64 inner solves
        _case("solve_256", "solve", n_e=256, M=10, p=3, sigma=0.25, L=0.3, degree=16, inner_rtol=1e-4,
              precision=64, precond="hsc", warm=False, rtol=1e-8),
        # the same solve with FP32 inner solves
        _case("solve_256_f32", "solve", n_e=256, M=10, p=3, sigma=0.25, L=0.3, degree=16, inner_rtol=1e-4,
              precision=32, precond="hsc", warm=False, rtol=1e-8),
        # the block Gauss-Seidel comparator with warm starts on an odd grid with Legendre chaos
        _case("bgs_75_legendre", "solve", n_e=75, M=5, p=3, sigma=0.3, L=0.5, family="legendre", degree=8,
              inner_rtol=1e-4, precision=64, precond="bgs", warm=True, rtol=1e-8),
        # forward solve and adjoint gradient of the 512^2 differentiation workload, 43M unknowns
        _case("grad_512", "grad", n_e=512, M=8, p=3, sigma=0.2, L=0.4, degree=16, inner_rtol=1e-4, rtol=1e-8),
        # sixteen uneven problems in one batch, FP32 inner solves and graph replay
        _case("batch_16", "batch", count=16, set=0, degree=16, max_grid=256, max_P=286, rtol=1e-8),
        # the lognormal solve on the 10 x 10 mesh of the published tables (CoV 100 %)
        _case("lognormal_10", "logn", n_e=10, M=4, p=4, cov=1.0, precond="hsc", rtol=1e-8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _chaos(rng, max_P, m_lo=2, m_hi=10, p_lo=1, p_hi=4):
    while True:
        M, p = rng.randint(m_lo, m_hi), rng.randint(p_lo, p_hi)
        if n_chaos(M, p) <= max_P:
            return M, p


def draw(rng):
    op = rng.choice(["matvec", "matvec", "inner", "hsc", "solve", "solve", "solve", "grad", "batch", "logn"])
    c = {"op": op, "family": rng.choice(["hermite", "legendre"]), "sigma": round(rng.uniform(0.1, 0.25), 4),
         "L": round(rng.uniform(0.3, 0.8), 4)}
    if op == "logn":
        M, p = _chaos(rng, 70, 1, 4, 1, 4)
        c.update(n_e=_log_int(rng, 6, 24), M=M, p=p, cov=round(rng.uniform(0.3, 1.0), 4), family="hermite",
                 precond=rng.choice(["hsc", "bgs", "mean"]), rtol=1e-8)
        return c
    if op == "batch":
        c.update(count=rng.randint(3, 16), set=rng.randrange(1 << 16), degree=rng.choice([8, 16]),
                 max_grid=rng.choice([64, 128]), max_P=286, family="hermite", rtol=1e-8)
        return c
    M, p = _chaos(rng, 286)
    c.update(n_e=_log_int(rng, 10, 256), M=M, p=p)
    if op in ("inner", "hsc", "solve", "grad"):
        c.update(degree=rng.choice([4, 8, 16]), inner_rtol=rng.choice([1e-4, 1e-6]))
    if op == "inner":
        c.update(ncols=rng.randint(1, n_chaos(M, p)))
    if op == "solve":
        c.update(precision=rng.choice([64, 32]), precond=rng.choice(["hsc", "bgs", "mean"]), warm=rng.random() < 0.25,
                 rtol=1e-8)
        if c["precision"] == 32:
            c["inner_rtol"] = 1e-4
    if op == "grad":
        c.update(rtol=1e-8)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

@functools.lru_cache(maxsize=32)
def _problem(n_e, M, p, sigma, L, family):
    return make_problem("case", n_e, M, p, sigma, L, family=family)


def _problem_of(case):
    return _problem(case["n_e"], case["M"], case["p"], case["sigma"], case["L"], case["family"])


@functools.lru_cache(maxsize=4)
def _batch_set(count, which, max_grid, max_P):
    grids = tuple(g for g in (32, 64, 128, 256) if g <= max_grid)
    return tuple(batch_problems(which, count, grids, max_P))


def _batch_of(case):
    return _batch_set(case["count"], case["set"], case["max_grid"], case["max_P"])


def _device():
    return torch.device("cuda", torch.cuda.current_device()) if torch.cuda.is_available() else torch.device("cpu")


def _normal(shape, seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, dtype=torch.float64, device=device)


def _load(P, n_e, seed, device):
    """The lumped load of f = 1 plus a seeded Gaussian bump, in the mean chaos block."""
    rng = np.random.default_rng(seed)
    bump = (rng.uniform(0.5, 2.0), rng.uniform(0.05, 0.2), rng.uniform(0.2, 0.8), rng.uniform(0.2, 0.8))
    F = torch.zeros((P, (n_e - 1) ** 2), dtype=torch.float64, device=device)
    F[0] = torch.from_numpy(nodal_rhs(n_e, bump) / (n_e * n_e))
    return F


def _inputs(case, seed):
    """The call's numeric inputs, on the GPU where there is one."""
    dev, op = _device(), case["op"]
    if op == "batch":
        return [_load(q.P, q.n_e, 1000 * seed + i, dev) for i, q in enumerate(_batch_of(case))]
    n, P = (case["n_e"] - 1) ** 2, n_chaos(case["M"], case["p"])
    if op in ("matvec", "hsc"):
        return _normal((P, n), seed, dev)
    if op == "inner":
        return _normal((case["ncols"], n), seed, dev)
    return _load(P, case["n_e"], seed, dev)


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------

def prepare(case, seed):
    from paper_1205_1864_amd.binding import LognormalOperator, Options, SGBatch, SGSolver
    op = case["op"]
    state = {"case": case, "x": _inputs(case, seed)}
    if op == "batch":
        state["solver"] = SGBatch(_batch_of(case), Options(inner_precision=32, cheb_degree=case["degree"],
                                                           precond="hsc", inner_maxit=2000))
    elif op == "logn":
        state["solver"] = LognormalOperator(_problem_of(case), mean=1.0, cov=case["cov"])
    else:
        opts = Options(inner_precision=case.get("precision", 64), cheb_degree=case.get("degree", 4),
                       inner_maxit=2000, precond=case.get("precond", "hsc"),
                       inner_rtol=case.get("inner_rtol", 1e-4), warm_start=case.get("warm", False))
        state["solver"] = SGSolver(_problem_of(case), opts)
        if op == "grad":
            wm, wv = qoi_weights(case["n_e"])
            state["wm"], state["wv"] = (torch.from_numpy(w).to(state["x"].device) for w in (wm, wv))
    return state


def run(state):
    case, s, x = state["case"], state["solver"], state["x"]
    op = case["op"]
    if op == "matvec":
        return {"Y": s.sg_matvec(x)}
    if op == "hsc":
        return {"Z": s.sg_apply_hsc(x)}
    if op == "inner":
        X, its = s.sg_inner_solve(x)
        return {"X": X, "its": its}
    if op == "solve":
        return {"U": s.sg_solve(x, rtol=case["rtol"], maxit=200)[0]}
    if op == "grad":
        U = s.sg_solve(x, rtol=case["rtol"], maxit=100)[0]
        lam = s.empty()
        Q, grad, _ = s.sg_adjoint_grad(U, state["wm"], state["wv"], rtol=case["rtol"], maxit=100, Lambda=lam)
        return {"U": U, "Lambda": lam, "Q": Q, "grad": grad}
    if op == "batch":
        return s.sg_batch_solve(x, rtol=case["rtol"], maxit=100)[0]
    return {"U": s.solve(x, rtol=case["rtol"], precond=case["precond"])[0]}


def _blocks(case):
    """Non-zero blocks of the global matrix: the diagonal and both neighbours per KL term."""
    M, p = case["M"], case["p"]
    return n_chaos(M, p) + (2 * M * math.comb(M + p - 1, M) if p else 0)


def work(case):
    """Inputs read once and outputs written once; the arithmetic of one product with the
    operator (of one mean-matrix product per column for the inner solves)."""
    op = case["op"]
    if op == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        for q in _batch_of(case):
            w = work({"op": "solve", "n_e": q.n_e, "M": q.M, "p": q.p})
            total = {k: total[k] + w[k] for k in total}
        return total
    ne, M, P = case["n_e"], case["M"], n_chaos(case["M"], case["p"])
    n = (ne - 1) ** 2
    if op == "inner":
        return {"bytes": 16.0 * n * case["ncols"], "flops": 18.0 * n * case["ncols"]}
    if op == "logn":
        # every pair of chaos functions couples through an element field
        return {"bytes": 16.0 * n * P + 8.0 * P * P * ne * ne, "flops": 32.0 * P * P * ne * ne}
    blocks = {"grad": 4}.get(op, 2)  # F, U, the adjoint solution and its right-hand side
    products = {"grad": 2}.get(op, 1)
    return {"bytes": 8.0 * blocks * n * P + 8.0 * M * ne * ne,
            "flops": products * ne * ne * (8.0 * _blocks(case) + 32.0 * P)}


# ---------------------------------------------------------------------------
# the same results in 64 bits from plain torch
# ---------------------------------------------------------------------------

def _multi_indices(M, p):
    """Graded by degree, descending lexicographic within a degree."""
    return [a for d in range(p + 1) for a in _compositions(M, d)]


def _compositions(M, d):
    if M == 0:
        if d == 0:
            yield ()
        return
    if M == 1:
        yield (d,)
        return
    for first in range(d, -1, -1):
        for rest in _compositions(M - 1, d - first):
            yield (first,) + rest


def _corners(U, ne):
    """The four corner values of every element, (P, ne, ne) views of the padded nodal field."""
    V = torch.zeros((U.shape[0], ne + 1, ne + 1), dtype=U.dtype, device=U.device)
    V[:, 1:ne, 1:ne] = U.reshape(U.shape[0], ne - 1, ne - 1)
    return V[:, :-1, :-1], V[:, :-1, 1:], V[:, 1:, :-1], V[:, 1:, 1:]


def _assemble(t, ne):
    """Sum of per-corner element vectors at the interior nodes."""
    P = t[0].shape[0]
    Y = torch.zeros((P, ne + 1, ne + 1), dtype=t[0].dtype, device=t[0].device)
    Y[:, :-1, :-1] += t[0]
    Y[:, :-1, 1:] += t[1]
    Y[:, 1:, :-1] += t[2]
    Y[:, 1:, 1:] += t[3]
    return Y[:, 1:ne, 1:ne].reshape(P, -1)


def _element(U, ne):
    """The unit-coefficient element matrix on each element: (4 u_c - u_e - u_e' - 2 u_opp) / 6."""
    a, b, c, d = _corners(U, ne)
    return ((4 * a - b - c - 2 * d) / 6, (4 * b - a - d - 2 * c) / 6, (4 * c - a - d - 2 * b) / 6,
            (4 * d - b - c - 2 * a) / 6)


class _System:
    """sum_k G_k (x) K_k and its mean block, in double precision."""

    def __init__(self, q, dev):
        self.ne, self.M, self.dev = q.n_e, q.M, dev
        self.alpha = _multi_indices(q.M, q.p)
        self.P = len(self.alpha)
        self.theta0 = q.theta0
        self.s, self.phi, self.sigma = q.s, torch.from_numpy(q.phi).to(dev), q.sigma
        self.a = [q.sigma * float(q.s[k]) * self.phi[k] for k in range(q.M)]
        row = {a: i for i, a in enumerate(self.alpha)}
        self.pairs = []
        for k in range(q.M):
            i, j, g = [], [], []
            for a, ia in row.items():
                up = a[:k] + (a[k] + 1,) + a[k + 1:]
                if up in row:
                    m = a[k]
                    w = math.sqrt(m + 1) if q.family == "hermite" else (m + 1) / math.sqrt((2 * m + 1) * (2 * m + 3))
                    i += [ia, row[up]]
                    j += [row[up], ia]
                    g += [w, w]
            G = torch.zeros((self.P, self.P), dtype=torch.float64)
            G[i, j] = torch.tensor(g, dtype=torch.float64)
            self.pairs.append(G.to(dev))
        self.level = [sum(a) for a in self.alpha]
        k = torch.arange(1, self.ne, dtype=torch.float64, device=dev)
        ang = torch.remainder(k[:, None] * k[None, :], 2 * self.ne)
        self.S = math.sqrt(2.0 / self.ne) * torch.sin(math.pi * ang / self.ne)
        c = torch.cos(math.pi * k / self.ne)
        self.lam = self.theta0 * (8 - 2 * c[:, None] - 2 * c[None, :] - 4 * c[:, None] * c[None, :]) / 3

    def apply_unit(self, U, field=None):
        t = _element(U, self.ne)
        return _assemble(t if field is None else [field * x for x in t], self.ne)

    def apply(self, U):
        Y = self.theta0 * self.apply_unit(U)
        for k in range(self.M):
            Y += self.apply_unit(self.pairs[k] @ U, self.a[k])
        return Y

    def couple(self, U, rows, cols):
        """The sub-block [rows, cols] (two levels) applied to U[cols]."""
        Y = 0
        for k in range(self.M):
            Y = Y + self.apply_unit(self.pairs[k][rows][:, cols] @ U, self.a[k])
        return Y

    def mean_inverse(self, R):
        nx = self.ne - 1
        V = torch.matmul(torch.matmul(R.reshape(-1, nx), self.S).reshape(-1, nx, nx).transpose(1, 2).reshape(-1, nx),
                         self.S).reshape(-1, nx, nx) / self.lam
        V = torch.matmul(torch.matmul(V.reshape(-1, nx), self.S).reshape(-1, nx, nx).transpose(1, 2).reshape(-1, nx),
                         self.S)
        return V.reshape(R.shape)

    def solve(self, F, rtol=1e-14, maxit=200):
        """Conjugate gradients preconditioned by the mean block, far past the calls' tolerance."""
        U, R = torch.zeros_like(F), F.clone()
        Z = self.mean_inverse(R)
        D, rz, fn = Z.clone(), torch.sum(R * Z), torch.linalg.norm(F)
        for _ in range(maxit):
            Q = self.apply(D)
            al = rz / torch.sum(D * Q)
            U += al * D
            R -= al * Q
            if float(torch.linalg.norm(R)) <= rtol * float(fn):
                break
            Z = self.mean_inverse(R)
            new = torch.sum(R * Z)
            D = Z + (new / rz) * D
            rz = new
        return U

    def pcg(self, B, degree, rtol, maxit):
        """Independent conjugate gradients on the mean block, one per row of B, preconditioned
        by ``degree`` updates of the Chebyshev iteration over the spectrum of D^-1 K_0; a row
        stops once its recursive residual passes."""
        ne, diag = self.ne, self.theta0 * 8.0 / 3.0
        c = math.cos(math.pi / ne)
        lo, hi = (8 - 4 * c - 4 * c * c) / 8, (8 + 4 * c * c) / 8
        theta, delta = 0.5 * (hi + lo), 0.5 * (hi - lo)

        def k0(V):
            return self.theta0 * self.apply_unit(V)

        def prec(R):
            S = R / diag
            W = S / theta
            Z = W.clone()
            s1 = theta / delta
            rho = 1.0 / s1
            for _ in range(1, degree):
                S = S - k0(W) / diag
                new = 1.0 / (2.0 * s1 - rho)
                W = (new * rho) * W + (2.0 * new / delta) * S
                Z = Z + W
                rho = new
            return Z

        X, R = torch.zeros_like(B), B.clone()
        bn = torch.linalg.norm(B, dim=1)
        its = torch.zeros(B.shape[0], dtype=torch.int64, device=B.device)
        live = bn > 0
        Z = prec(R)
        D, gam = Z.clone(), torch.sum(R * Z, 1)
        for it in range(maxit):
            if not bool(live.any()):
                break
            Q = k0(D)
            al = torch.where(live, gam / torch.sum(D * Q, 1), torch.zeros_like(gam))
            X += al[:, None] * D
            R -= al[:, None] * Q
            its[live] = it + 1
            live = live & ~(torch.linalg.norm(R, dim=1) <= rtol * bn)
            Z = prec(R)
            new = torch.sum(R * Z, 1)
            D = Z + torch.where(live, new / gam, torch.zeros_like(gam))[:, None] * D
            gam = new
        return X, its

    def hsc(self, R, solve):
        """Algorithm 1: pre-corrections down the levels, the mean problem, post-corrections up."""
        lev = torch.tensor(self.level, device=self.dev)
        at = [torch.nonzero(lev == d).flatten() for d in range(max(self.level) + 1)]
        r, u = R.clone(), torch.zeros_like(R)
        for d in range(len(at) - 1, 0, -1):
            r[at[d - 1]] -= self.couple(solve(r[at[d]]), at[d - 1], at[d])
        u[at[0]] = solve(r[at[0]])
        for d in range(1, len(at)):
            u[at[d]] = solve(r[at[d]] - self.couple(u[at[d - 1]], at[d], at[d - 1]))
        return u


def _lognormal(case, q, F, dev):
    """A U = F for the coefficient exp(g) of mean 1, with A_ab = K(E[k psi_a psi_b]), by
    conjugate gradients preconditioned by the unit-coefficient mean block."""
    sg2 = math.log1p(case["cov"] ** 2)
    mu = -0.5 * sg2
    alpha = _multi_indices(q.M, q.p)
    g = math.sqrt(sg2) * torch.from_numpy(np.asarray(q.s)[:, None, None] * q.phi).to(dev)
    # E[exp(g xi) psi_a psi_b] = exp(g^2 / 2) sum_i E[psi_i psi_a psi_b] g^i / sqrt(i!) per variable
    one = {}
    for k in range(q.M):
        for a in range(q.p + 1):
            for b in range(q.p + 1):
                t = torch.zeros_like(g[k])
                for i in range(abs(a - b), a + b + 1, 2):
                    s = (a + b + i) // 2
                    tri = math.sqrt(math.factorial(a) * math.factorial(b) * math.factorial(i)) / (
                        math.factorial(s - a) * math.factorial(s - b) * math.factorial(s - i))
                    t = t + tri / math.sqrt(math.factorial(i)) * g[k] ** i
                one[k, a, b] = t
    base = torch.exp(mu + 0.5 * (g * g).sum(0))
    P, ne = len(alpha), q.n_e
    C = torch.empty((P, P, ne, ne), dtype=torch.float64, device=dev)
    for i, a in enumerate(alpha):
        for j, b in enumerate(alpha):
            f = base
            for k in range(q.M):
                f = f * one[k, a[k], b[k]]
            C[i, j] = f
    unit = _System(make_problem("mean", ne, 0, 0, 0.0, 1.0), dev)

    def apply(U):
        t = [torch.stack([(C[i] * x).sum(0) for i in range(P)]) for x in _element(U, ne)]
        return _assemble(t, ne)

    U, R = torch.zeros_like(F), F.clone()
    Z = unit.mean_inverse(R)
    D, rz, fn = Z.clone(), torch.sum(R * Z), float(torch.linalg.norm(F))
    for _ in range(3000):
        Q = apply(D)
        al = rz / torch.sum(D * Q)
        U += al * D
        R -= al * Q
        if float(torch.linalg.norm(R)) <= 1e-13 * fn:
            break
        Z = unit.mean_inverse(R)
        new = torch.sum(R * Z)
        D = Z + (new / rz) * D
        rz = new
    return U


def exact(case, seed):
    dev, op, x = _device(), case["op"], _inputs(case, seed)
    if op == "batch":
        return [_System(q, dev).solve(f) for q, f in zip(_batch_of(case), x)]
    q = _problem_of(case)
    if op == "logn":
        return {"U": _lognormal(case, q, x, dev)}
    S = _System(q, dev)
    if op == "matvec":
        return {"Y": S.apply(x)}
    if op == "inner":
        X, its = S.pcg(x, case["degree"], case["inner_rtol"], 2000)
        return {"X": X, "its": its}
    if op == "hsc":
        return {"Z": S.hsc(x, lambda B: S.pcg(B, case["degree"], case["inner_rtol"], 2000)[0])}
    U = S.solve(x)
    if op == "solve":
        return {"U": U}
    wm, wv = (torch.from_numpy(w).to(dev) for w in qoi_weights(case["n_e"]))
    Q = float(torch.dot(wm, U[0]) + (wv * U[1:] ** 2).sum())
    G = 2 * wv * U
    G[0] = wm
    lam = S.solve(G)
    grad = [-float(torch.sum(lam * S.apply_unit(U)))]
    for k in range(q.M):
        grad.append(-q.sigma * float(torch.sum(lam * S.apply_unit(S.pairs[k] @ U, S.phi[k]))))
    return {"U": U, "Lambda": lam, "Q": Q, "grad": np.array(grad)}
