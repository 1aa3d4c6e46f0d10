"""Algorithmic bytes of the inner launches in the sine basis: every transform pass
and the iteration read and write a vector per column. Columns of up to 64 rows are
transformed within the iteration's launch, where both directions are one pass."""

import pytest

pytestmark = pytest.mark.gpu

from sg_inputs import make_problem  # noqa: E402


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("n_e,cold,warm", [(20, 6, 9), (65, 6, 9), (66, 10, 15), (130, 10, 15)])
def test_inner_bytes_follow_the_launches(n_e, cold, warm, prec):
    from paper_1205_1864_amd import binding as b
    prob = make_problem("bytes", n_e, 2, 1, 0.2, 0.5)
    print(f"inner bytes n_e={n_e} FP{prec}", flush=True)
    F = b.to_device_block(prob.load_block())
    for ws in (False, True):
        solver = b.SGSolver(prob, b.Options(inner_precision=prec, inner_maxit=5, inner_rtol=0.0, warm_start=ws))
        _, st = solver.sg_solve(F, rtol=1e-14, maxit=1)
        solver.close()
        assert st["outer_it"] == 1 and st["inner_launches"] == 3
        # two columns down, one for the mean, two up (the warm ones)
        vectors = 3 * cold + 2 * (warm if ws else cold)
        assert st["inner_bytes"] == vectors * prob.n * (prec // 8)
