"""Coupling products of launches large enough for the strip kernel's automatic rows of
both directions, against the oracle: six rows a wave towards the lower level (300^2: from
some 6000 waves on), four towards the higher one."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import sg  # noqa: E402
from sg_inputs import make_problem, random_block  # noqa: E402


# 299 rows are no multiple of 4 or 6; 28 rows of level 2 make 7000 waves of six, 21 make 5250
@pytest.mark.parametrize("M", [7, 6])
def test_large_coupling_products(M):
    from paper_1205_1864_amd import binding as b
    prob = make_problem("strip", 300, M, 3, 0.2, 0.5)
    s = sg.build_system(prob)
    print(f"large couplings M={M}", flush=True)
    solver = b.SGSolver(prob)
    U = random_block(prob.P, prob.n, seed=M)
    Ud = b.to_device_block(U)
    lo, hi, top = s.off[2], s.off[3], s.off[4]
    for direction in (0, 1):
        R = random_block(prob.P, prob.n, seed=10 + direction)
        Rg = solver.sg_coupling(3, direction, b.to_device_block(R), Ud).cpu().numpy()
        Ro = R.T.copy()
        if direction == 0:
            Ro[:, lo:hi] -= sg.level_block(s, slice(lo, hi), slice(hi, top))(U.T[:, hi:top])
        else:
            Ro[:, hi:top] -= sg.level_block(s, slice(hi, top), slice(lo, hi))(U.T[:, lo:hi])
        assert np.linalg.norm(Rg - Ro.T) <= 1e-13 * np.linalg.norm(Ro)
    solver.close()
