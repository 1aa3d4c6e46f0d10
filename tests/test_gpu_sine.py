"""The inner solver in the sine basis (automatic tiles) against the oracle's PCG
and against the tiled solver, at the edges of its tiles, of its transform
variants and of the number of blocks that share a column."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import krylov, sg  # noqa: E402
from sg_inputs import make_problem, random_block  # noqa: E402


def _solver(prob, **kw):
    from paper_1205_1864_amd import binding as b
    return b.SGSolver(prob, b.Options(**kw))


# n_e and what changes there: the smallest grid; one and two 16-mode tiles per
# parity (33 / 34); one and five launches a solve (65 / 66); 3, 4 and 5 tiles (65, 97, 130), 5, 8, 11 and 23 slots per
# thread; two blocks per column (131, 200: 14 and 27 slots), three (256, 257: an even
# and an odd number of modes per parity; 258), ten to twelve (512, 514, 515). Transforms
# in four products from 34 on where n_e is even (n_e / 2 odd: 34, 66, 130, 258, 514;
# even: 36, 200, 256, 512), in two elsewhere; more than sixteen tiles from 514 on
SIZES = [3, 4, 5, 32, 33, 34, 36, 65, 66, 97, 130, 131, 200, 256, 257, 258, 512, 514, 515]


@pytest.mark.parametrize("prec,tol", [(64, 1e-11), (32, 2e-5)])
@pytest.mark.parametrize("n_e", SIZES)
def test_fixed_iterations_match_oracle(n_e, prec, tol):
    """Iterates after a fixed number of iterations, to the tolerances of the tiled
    solver's own tests (rounding of a short iteration sequence)."""
    from paper_1205_1864_amd import binding as b
    prob = make_problem("sine", n_e, 2, 1, 0.2, 0.5)
    K0 = sg.build_system(prob).K[0]
    B = random_block(3, prob.n, seed=n_e)
    B[1] = 0.0
    for degree in (1, 6):
        # before the residual reaches zero on the smallest grids, above the cap that takes the tiles on the largest
        its = 8 if n_e > 500 else min(5, n_e - 2)
        print(f"sine n_e={n_e} FP{prec} degree={degree}", flush=True)
        solver = _solver(prob, inner_precision=prec, cheb_degree=degree, inner_maxit=its, inner_rtol=0.0)
        X, it = solver.sg_inner_solve(b.to_device_block(B))
        solver.close()
        X = X.cpu().numpy()
        Xo = krylov.pcg_columns(K0, B.T, krylov.make_chebyshev(K0, n_e, prob.theta0, degree), 0.0, its).T
        assert list(it) == [its, 0, its]
        assert np.all(X[1] == 0.0)
        for c in (0, 2):
            assert np.linalg.norm(X[c] - Xo[c]) <= tol * np.linalg.norm(Xo[c])


@pytest.mark.parametrize("prec,tol", [(64, 1e-11), (32, 1e-4)])
@pytest.mark.parametrize("n_e,ncols", [(12, 120), (47, 35), (101, 20), (201, 90), (256, 90), (300, 35)])
def test_solves_match_tiled_solver(n_e, ncols, prec, tol):
    """Solves to a tolerance, more columns than groups of blocks among them, cold
    and (through a warm-started action) warm: the tiled solver's counts and results.
    A column with a NaN ends with the same count and no effect on the others. The
    FP32 bound is that of one inner tolerance."""
    import torch
    from paper_1205_1864_amd import binding as b
    prob = make_problem("sine", n_e, 7, 3, 0.2, 0.5)
    assert prob.P == 120
    B = random_block(ncols, prob.n, seed=n_e)
    B[ncols // 2, 3] = np.nan
    R = random_block(prob.P, prob.n, seed=n_e + 1) if n_e <= 101 else None
    out = []
    for tile in (0, 32):
        print(f"sine against tiles n_e={n_e} ncols={ncols} FP{prec} tile={tile}", flush=True)
        solver = _solver(prob, inner_precision=prec, cheb_degree=8, inner_maxit=500, inner_rtol=1e-4, tile=tile,
                         warm_start=True)
        X, it = solver.sg_inner_solve(b.to_device_block(B))
        Z = solver.sg_apply_hsc(b.to_device_block(R)) if R is not None else torch.zeros(1, device="cuda")
        out.append((X.cpu().numpy(), list(it), Z.cpu().numpy()))
        solver.close()
    (X, it, Z), (Xt, itt, Zt) = out
    assert it[ncols // 2] == itt[ncols // 2] == 0
    assert np.array_equal(X[ncols // 2], Xt[ncols // 2], equal_nan=True)
    for c in range(ncols):
        if c != ncols // 2:
            assert abs(it[c] - itt[c]) <= (0 if prec == 64 else 1)
            assert np.linalg.norm(X[c] - Xt[c]) <= tol * np.linalg.norm(Xt[c])
    if R is not None:
        assert np.linalg.norm(Z - Zt) <= tol * np.linalg.norm(Zt)


def test_more_columns_than_a_grid_dimension():
    """A chaos of more than 65535 functions on the smallest grid: one launch takes every column."""
    from paper_1205_1864_amd import binding as b
    prob = make_problem("sine", 3, 0, 0, 0.2, 0.5)
    prob.M, prob.p = 44, 4
    prob.s = np.zeros(44)
    prob.phi = np.zeros((44, 3, 3))
    print("sine many columns", flush=True)
    solver = _solver(prob, inner_maxit=50, inner_rtol=1e-13)
    assert solver.P > 65535
    B = random_block(solver.P, prob.n, seed=1)
    X, it = solver.sg_inner_solve(b.to_device_block(B))
    solver.close()
    K0 = sg.build_system(make_problem("k0", 3, 0, 0, 0.0, 0.5)).K[0].toarray()
    assert np.max(np.abs(X.cpu().numpy() @ K0 - B)) <= 1e-11 * np.max(np.abs(B))
    assert np.all(it > 0)


@pytest.mark.parametrize("prec,pc,warm", [(64, "hsc", True), (32, "bgs", False)])
def test_batch_classes_match_single_solves(prec, pc, warm):
    """A batch whose members differ in slots per thread and blocks per column (one,
    two and six): each member as its own solve, to the batch tests' tolerances."""
    from paper_1205_1864_amd import binding as b
    probs = [make_problem(f"c{i}", n_e, M, p, 0.2, 0.5)
             for i, (n_e, M, p) in enumerate([(20, 3, 2), (70, 2, 2), (130, 2, 1), (300, 2, 2), (101, 1, 2)])]
    opts = b.Options(inner_precision=prec, precond=pc, cheb_degree=8, inner_rtol=1e-4, warm_start=warm)
    F = [b.to_device_block(pr.load_block()) for pr in probs]
    print(f"sine batch classes FP{prec} {pc} warm={warm}", flush=True)
    batch = b.SGBatch(probs, opts)
    U, stats, info = batch.sg_batch_solve(F, rtol=1e-8, maxit=100)
    assert info["rc"] == 0
    for i, pr in enumerate(probs):
        single = b.SGSolver(pr, opts)
        Us, ss = single.sg_solve(F[i], rtol=1e-8, maxit=100)
        single.close()
        assert abs(stats[i]["outer_it"] - ss["outer_it"]) <= (0 if prec == 64 else 1)
        assert float((U[i] - Us).norm() / Us.norm()) <= (1e-11 if prec == 64 else 1e-7)
    batch.close()
