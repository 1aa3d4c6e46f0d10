"""The library tells which solver its inner launches take: the sine basis (0),
banded (32) or square (16) tiles, by the options, the grid and the tuners."""

import pytest

pytestmark = pytest.mark.gpu

from sg_inputs import make_problem  # noqa: E402


@pytest.mark.parametrize("n_e,maxit,tile,kind", [
    (20, 1000, 0, 0), (20, 1000, 32, 32), (20, 1000, 16, 16),
    # the cap below which few iterations go to the tiles: nx / 176
    (300, 2, 0, 0), (300, 1, 0, 32), (1025, 6, 0, 0), (1025, 5, 0, 32), (1026, 1000, 0, 32),
])
def test_inner_kind_follows_the_options(n_e, maxit, tile, kind):
    from paper_1205_1864_amd import binding as b
    prob = make_problem("kind", n_e, 0, 0, 0.2, 0.5)
    opts = dict(inner_maxit=maxit, tile=tile)
    solver = b.SGSolver(prob, b.Options(**opts))
    assert solver.inner_kind() == kind
    solver.set_opts(b.Options(inner_maxit=maxit, tile=16))
    assert solver.inner_kind() == 16
    solver.set_opts(b.Options(**opts))
    assert solver.inner_kind() == kind
    solver.close()


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


@pytest.mark.parametrize("tile,n_e,kind", [(0, 20, 0), (32, 20, 32), (16, 20, 16), (0, 1026, 32)])
def test_batch_inner_kind(tile, n_e, kind):
    from paper_1205_1864_amd import binding as b
    probs = [make_problem(f"k{i}", g, 1, 1, 0.2, 0.5) for i, g in enumerate((12, n_e))]
    batch = b.SGBatch(probs, b.Options(inner_precision=32, tile=tile))
    assert batch.inner_kind() == kind
    batch.close()
