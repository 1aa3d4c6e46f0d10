"""The tiled inner solver, asked for by name or by an iteration cap that the sine
basis does not serve: launch schedules, automatic band heights, warm starts and
ragged launches. Each test asks the library which solver it runs."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hsc, krylov, sg  # noqa: E402
from sg_inputs import make_problem, named_problem, random_block  # noqa: E402


def _b():
    from paper_1205_1864_amd import binding
    return binding


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("degree", [16, 3])
def test_banded_schedules_bitwise_equal(prec, degree, monkeypatch):
    """The automatic grid, a cap of 128 blocks and whole columns per block run the same
    arithmetic per column: equal bits and counts for the 220 top-level columns of
    256^2, after twelve iterations and to a tolerance, the former as the oracle's."""
    b = _b()
    prob = named_problem("scale")
    B = random_block(220, prob.n, seed=3)
    Bd = b.to_device_block(B)
    res = []
    for mb in ("0", "128", "-1"):
        print(f"banded schedule max_blocks={mb} prec={prec} degree={degree}", flush=True)
        monkeypatch.setenv("SGPC_PCG_MAX_BLOCKS", mb)
        opts = dict(inner_precision=prec, cheb_degree=degree, tile=32)
        solver = b.SGSolver(prob, b.Options(**opts, inner_maxit=12, inner_rtol=0.0))
        assert solver.inner_kind() == 32
        X12, its12 = solver.sg_inner_solve(Bd)
        solver.set_opts(b.Options(**opts, inner_maxit=2000, inner_rtol=1e-4))
        Xt, itst = solver.sg_inner_solve(Bd)
        res.append((X12.cpu(), list(its12), Xt.cpu(), list(itst)))
        solver.close()
    for X12, its12, Xt, itst in res[1:]:
        assert bool((X12 == res[0][0]).all()) and its12 == res[0][1]
        assert bool((Xt == res[0][2]).all()) and itst == res[0][3]
    assert all(i == 12 for i in res[0][1])
    K0 = sg.build_system(prob).K[0]
    cols = [0, 97, 219]
    Xo = krylov.pcg_columns(K0, B[cols].T, krylov.make_chebyshev(K0, prob.n_e, prob.theta0, degree), 0.0, 12).T
    tol = 1e-11 if prec == 64 else 2e-5
    for j, c in enumerate(cols):
        assert np.linalg.norm(res[0][0][c].numpy() - Xo[j]) <= tol * np.linalg.norm(Xo[j])


# automatic tiles (tile = 0) with a cap below nx / 176: 64-row bands of a few columns (300, five per
# tile column), the 128-row bands of ten columns of 255 x 255 at degree 16 (the FP32 kernel's middle
# height), several bands and a ragged last one (512), and the first grid past the sine basis
@pytest.mark.parametrize("prec,tol", [(64, 1e-11), (32, 2e-5)])
@pytest.mark.parametrize("n_e,ncols,degree,maxit", [(300, 3, 2, 1), (300, 3, 8, 1), (300, 3, 16, 1), (256, 10, 16, 1),
                                                    (512, 3, 8, 2), (1026, 3, 8, 6)])
def test_automatic_bands(n_e, ncols, degree, maxit, prec, tol):
    b = _b()
    prob = make_problem("bands", n_e, 3, 2, 0.2, 0.5)
    print(f"automatic bands n_e={n_e} ncols={ncols} degree={degree} prec={prec}", flush=True)
    solver = b.SGSolver(prob, b.Options(inner_precision=prec, cheb_degree=degree, inner_maxit=maxit, inner_rtol=0.0))
    assert solver.inner_kind() == 32
    B = random_block(ncols, prob.n, seed=n_e + degree)
    X, its = solver.sg_inner_solve(b.to_device_block(B))
    solver.close()
    K0 = sg.build_system(make_problem("k0", n_e, 0, 0, 0.0, 0.5)).K[0]
    Xo = krylov.pcg_columns(K0, B.T, krylov.make_chebyshev(K0, n_e, prob.theta0, degree), 0.0, maxit).T
    assert list(its) == [maxit] * ncols
    X = X.cpu().numpy()
    for c in range(ncols):
        assert np.linalg.norm(X[c] - Xo[c]) <= tol * np.linalg.norm(Xo[c])


@pytest.mark.parametrize("prec,tol", [(64, 1e-11), (32, 1e-4)])
@pytest.mark.parametrize("n_e", [4, 52, 130])
@pytest.mark.parametrize("degree", [1, 2, 4, 8])
def test_banded_warm_fixed_iterations(prec, tol, n_e, degree):
    """Three iterations a solve, the up sweep from the down sweep's values: the oracle's
    Algorithm 1 with the same inner PCG from the same guesses."""
    b = _b()
    prob = make_problem("warm", n_e, 2, 2, 0.3, 0.5)
    s = sg.build_system(prob)
    solver = b.SGSolver(prob, b.Options(inner_precision=prec, cheb_degree=degree, inner_maxit=3, inner_rtol=0.0,
                                        tile=32, warm_start=True))
    assert solver.inner_kind() == 32
    R = random_block(prob.P, prob.n, seed=12)
    Z = solver.sg_apply_hsc(b.to_device_block(R)).cpu().numpy()
    solver.close()
    Zo = hsc.hsc_apply(s, R.T, hsc.PCGMeanSolver(s, 0.0, 3, degree), warm=True).T
    assert np.linalg.norm(Z - Zo) <= tol * np.linalg.norm(Zo)
    if prec == 64 and n_e >= 52:
        Zc = hsc.hsc_apply(s, R.T, hsc.PCGMeanSolver(s, 0.0, 3, degree)).T
        assert np.linalg.norm(Z - Zc) > 1e3 * tol * np.linalg.norm(Zo)


@pytest.mark.parametrize("prec,pc,warm", [(64, "hsc", False), (32, "hsc", True), (64, "bgs", True), (32, "bgs", False),
                                         (64, "mean", False)])
def test_banded_batch_matches_single_solves(prec, pc, warm):
    """Ragged banded launches, cold and warm, against each member's own banded solve, to
    the batch tests' tolerances."""
    b = _b()
    probs = [make_problem(f"t{i}", n_e, M, p, 0.2, 0.5)
             for i, (n_e, M, p) in enumerate([(16, 4, 2), (64, 3, 3), (21, 2, 1), (128, 2, 2), (200, 1, 2)])]
    opts = b.Options(inner_precision=prec, precond=pc, cheb_degree=8, inner_rtol=1e-4, warm_start=warm, tile=32)
    print(f"banded batch FP{prec} {pc} warm={warm}", flush=True)
    batch = b.SGBatch(probs, opts)
    assert batch.inner_kind() == 32
    F = [b.to_device_block(pr.load_block()) for pr in probs]
    U, stats, info = batch.sg_batch_solve(F, rtol=1e-8, maxit=100)
    assert info["rc"] == 0
    for i, pr in enumerate(probs):
        single = b.SGSolver(pr, opts)
        assert single.inner_kind() == 32
        Us, ss = single.sg_solve(F[i], rtol=1e-8, maxit=100)
        single.close()
        assert stats[i]["true_relres"] <= 1.05e-8
        assert abs(stats[i]["outer_it"] - ss["outer_it"]) <= (0 if prec == 64 else 1)
        assert float((U[i] - Us).norm() / Us.norm()) <= (1e-11 if prec == 64 else 1e-7)
    batch.close()
