"""The sine-basis solver's longest transforms (more than sixteen pairs of product
tiles, strips of 16 lines, up to 39 blocks a column), alone and in a ragged launch
beside short ones, and the grid on which the tiles take over."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import krylov, sg  # noqa: E402
from sg_inputs import make_problem, random_block  # noqa: E402


# two products of 32 tiles a transform, the longest four of 16 (n_e even), the longest of
# all, and past the sine basis
@pytest.mark.parametrize("prec,tol", [(64, 1e-11), (32, 2e-5)])
@pytest.mark.parametrize("n_e,kind", [(1023, 0), (1024, 0), (1025, 0), (1026, 32)])
def test_fixed_iterations_match_oracle(n_e, kind, prec, tol):
    """To the tolerances of the shorter transforms' and the tiled solver's tests."""
    from paper_1205_1864_amd import binding as b
    prob = make_problem("long", n_e, 2, 1, 0.2, 0.5)
    K0 = sg.build_system(make_problem("k0", n_e, 0, 0, 0.0, 0.5)).K[0]
    B = random_block(3, prob.n, seed=n_e)
    B[1] = 0.0
    its = 8
    for degree in (1, 6):
        print(f"long sine n_e={n_e} FP{prec} degree={degree}", flush=True)
        solver = b.SGSolver(prob, b.Options(inner_precision=prec, cheb_degree=degree, inner_maxit=its, inner_rtol=0.0))
        assert solver.inner_kind() == kind
        X, it = solver.sg_inner_solve(b.to_device_block(B))
        solver.close()
        X = X.cpu().numpy()
        Xo = krylov.pcg_columns(K0, B.T, krylov.make_chebyshev(K0, n_e, prob.theta0, degree), 0.0, its).T
        assert list(it) == [its, 0, its]
        assert np.all(X[1] == 0.0)
        for c in (0, 2):
            assert np.linalg.norm(X[c] - Xo[c]) <= tol * np.linalg.norm(Xo[c])


@pytest.mark.parametrize("prec,pc,warm", [(64, "hsc", True), (32, "bgs", False)])
@pytest.mark.parametrize("longest", [600, 1025])
def test_long_beside_short_in_one_batch(longest, prec, pc, warm):
    """A member with two rounds of product tiles a wave beside very short ones: each as
    its own solve, to the batch tests' tolerances."""
    from paper_1205_1864_amd import binding as b
    probs = [make_problem(f"l{i}", n_e, M, p, 0.2, 0.5)
             for i, (n_e, M, p) in enumerate([(3, 2, 1), (longest, 1, 1), (20, 2, 2), (130, 1, 1), (514, 1, 1)])]
    opts = b.Options(inner_precision=prec, precond=pc, cheb_degree=8, inner_rtol=1e-4, warm_start=warm)
    F = [b.to_device_block(pr.load_block()) for pr in probs]
    print(f"long batch {longest} FP{prec} {pc} warm={warm}", flush=True)
    batch = b.SGBatch(probs, opts)
    assert batch.inner_kind() == 0
    U, stats, info = batch.sg_batch_solve(F, rtol=1e-8, maxit=100)
    assert info["rc"] == 0
    for i, pr in enumerate(probs):
        single = b.SGSolver(pr, opts)
        Us, ss = single.sg_solve(F[i], rtol=1e-8, maxit=100)
        single.close()
        assert stats[i]["true_relres"] <= 1.05e-8
        assert abs(stats[i]["outer_it"] - ss["outer_it"]) <= (0 if prec == 64 else 1)
        assert float((U[i] - Us).norm() / Us.norm()) <= (1e-11 if prec == 64 else 1e-7)
    batch.close()
