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


@pytest.mark.parametrize("tile,n_e,kind", [(0, 20, 0), (32, 20, 32), (16, 20, 16), (0, 1026, 32)])
def test_batch_inner_kind(tile, n_e, kind):
    from paper_1205_1864_amd import binding as b
    probs = [make_problem(f"k{i}", g, 1, 1, 0.2, 0.5) for i, g in enumerate((12, n_e))]
    batch = b.SGBatch(probs, b.Options(inner_precision=32, tile=tile))
    assert batch.inner_kind() == kind
    batch.close()
