"""The library tells which solver its inner launches take: the sine basis (0),
banded (32) or square (16) tiles, by the options, the grid and the tuners."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import hsc, sg  # noqa: E402
from sg_inputs import make_problem, random_block  # noqa: E402


@pytest.mark.parametrize("n_e,M,maxit,tile,kind", [
    (20, 2, 1000, 0, 0), (20, 2, 1000, 32, 32), (20, 2, 1000, 16, 16),
    # the cap below which few iterations go to the tiles: nx / 176 for three columns
    (300, 2, 2, 0, 0), (300, 2, 1, 0, 32), (1025, 2, 6, 0, 0), (1025, 2, 5, 0, 32), (1026, 2, 1000, 0, 32),
    # (nx + 100) / 176 for two, and for one nx / 110 in two products a transform, (nx + 100) / 176 in four
    (1025, 1, 7, 0, 0), (1025, 1, 6, 0, 32), (1025, 0, 10, 0, 0), (1025, 0, 9, 0, 32), (1024, 0, 7, 0, 0),
    (1024, 0, 6, 0, 32), (129, 0, 1, 0, 0), (130, 0, 2, 0, 0), (130, 0, 1, 0, 32),
])
def test_inner_kind_follows_the_options(n_e, M, maxit, tile, kind):
    from paper_1205_1864_amd import binding as b
    prob = make_problem("kind", n_e, M, 1 if M else 0, 0.2, 0.5)
    opts = dict(inner_maxit=maxit, tile=tile)
    solver = b.SGSolver(prob, b.Options(**opts))
    assert solver.inner_kind() == kind
    solver.set_opts(b.Options(inner_maxit=maxit, tile=16))
    assert solver.inner_kind() == 16
    solver.set_opts(b.Options(**opts))
    assert solver.inner_kind() == kind
    solver.close()


@pytest.mark.parametrize("prec,tol", [(64, 1e-11), (32, 1e-4)])
@pytest.mark.parametrize("warm", [False, True])
def test_an_action_on_both_solvers(warm, prec, tol):
    """Two iterations a solve at 300^2: the mean's one column on tiles, the three of level
    one in the sine basis (10 n w of bytes a column, (9 its + 6) n w on tiles, warm more);
    the oracle's Algorithm 1 with the same inner PCG, to the fixed-iteration tolerances."""
    from paper_1205_1864_amd import binding as b
    prob = make_problem("both", 300, 3, 1, 0.3, 0.5)
    s = sg.build_system(prob)
    print(f"both solvers warm={warm} FP{prec}", flush=True)
    solver = b.SGSolver(prob, b.Options(inner_precision=prec, cheb_degree=4, inner_maxit=2, inner_rtol=0.0,
                                        warm_start=warm))
    R = random_block(prob.P, prob.n, seed=12)
    Z = solver.sg_apply_hsc(b.to_device_block(R)).cpu().numpy()
    Zo = hsc.hsc_apply(s, R.T, hsc.PCGMeanSolver(s, 0.0, 2, 4), warm=warm).T
    assert np.linalg.norm(Z - Zo) <= tol * np.linalg.norm(Zo)
    _, st = solver.sg_solve(b.to_device_block(prob.load_block()), rtol=1e-14, maxit=1)
    solver.close()
    assert st["inner_launches"] == 3
    assert st["inner_bytes"] == (3 * 10 + 3 * (15 if warm else 10) + 9 * 2 + 6) * prob.n * (prec // 8)


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("tile,kinds,candidates", [(0, (0,), 7), (32, (16, 32), 6), (16, (16, 32), 6)])
def test_autotune_stays_within_the_tiles_asked_for(tile, kinds, candidates, prec):
    """A caller of square or banded tiles is moved between those two, three block
    counts each; the sine basis is one candidate more with automatic tiles (on this
    grid more than ten times faster than either, so it is the pick)."""
    from paper_1205_1864_amd import binding as b
    prob = make_problem("kind", 100, 3, 2, 0.2, 0.5)
    print(f"autotune tile={tile} FP{prec}", flush=True)
    solver = b.SGSolver(prob, b.Options(inner_precision=prec, cheb_degree=8, tile=tile))
    rep = solver.sg_autotune(2)
    assert rep["candidates"] == candidates and rep["pcg_tile"] in (16, 32)
    assert solver.inner_kind() in kinds
    F = b.to_device_block(prob.load_block())
    U, st = solver.sg_solve(F, rtol=1e-8, maxit=100)
    assert st["rc"] == 0 and st["true_relres"] <= 1.05e-8
    solver.set_opts(b.Options(inner_precision=prec, cheb_degree=8))
    assert solver.inner_kind() == 0
    solver.close()


@pytest.mark.parametrize("prec,pc", [(64, "hsc"), (32, "bgs"), (64, "mean")])
@pytest.mark.parametrize("n_e,M,p", [(40, 5, 3), (130, 4, 2), (20, 2, 0)])
def test_tuned_operator_and_couplings(n_e, M, p, prec, pc):
    """The operator's tuner reports a kernel that exists and a schedule with which the
    operator and the coupling products are the oracle's (chaos without a coupling too)."""
    from paper_1205_1864_amd import binding as b
    prob = make_problem("tune", n_e, M, p, 0.2, 0.5)
    s = sg.build_system(prob)
    print(f"operator tuner n_e={n_e} FP{prec} {pc}", flush=True)
    solver = b.SGSolver(prob, b.Options(inner_precision=prec, precond=pc))
    rep = solver.sg_autotune(1)
    assert rep["mv_variant"] in (3, 4) and rep["mv_ms"] > 0 and rep["candidates"] >= 5
    assert rep["mv_param"] in (0, 200, 400, 600, 800) if rep["mv_variant"] == 3 else rep["mv_param"] > 0
    U = random_block(prob.P, prob.n, seed=4)
    Ud = b.to_device_block(U)
    Yo = sg.matvec(s, U.T.copy()).T
    assert np.linalg.norm(solver.sg_matvec(Ud).cpu().numpy() - Yo) <= 1e-12 * np.linalg.norm(Yo)
    for level in range(1, p + 1):
        lo, hi = s.off[level], s.off[level + 1]
        below = s.off[level - 1]
        R = random_block(prob.P, prob.n, seed=level)
        Ro = R.T.copy()
        Ro[:, below:lo] -= sg.level_block(s, slice(below, lo), slice(lo, hi))(U.T[:, lo:hi])
        Rg = solver.sg_coupling(level, 0, b.to_device_block(R), Ud).cpu().numpy()
        assert np.linalg.norm(Rg - Ro.T) <= 1e-13 * np.linalg.norm(Ro)
    solver.close()


@pytest.mark.parametrize("tile,n_e,kind", [(0, 20, 0), (32, 20, 32), (16, 20, 16), (0, 1026, 32)])
def test_batch_inner_kind(tile, n_e, kind):
    from paper_1205_1864_amd import binding as b
    probs = [make_problem(f"k{i}", g, 1, 1, 0.2, 0.5) for i, g in enumerate((12, n_e))]
    batch = b.SGBatch(probs, b.Options(inner_precision=32, tile=tile))
    assert batch.inner_kind() == kind
    batch.close()
