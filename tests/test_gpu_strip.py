"""The strip kernel of the SG operator and its coupling products against the
oracle, at the edges of its strips (62 node columns) and row groups."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import sg  # noqa: E402
from sg_inputs import make_problem, random_block  # noqa: E402


# one node, one strip exactly full (62 columns), one more, two strips full (124)
# and one more, and a grid of four strips whose launches fill the device
@pytest.mark.parametrize("rows", [0, 2, 4, 6, 8])
@pytest.mark.parametrize("n_e", [3, 6, 62, 63, 64, 125, 126, 190])
def test_strip_operator_and_couplings(n_e, rows, monkeypatch):
    from paper_1205_1864_amd import binding as b
    monkeypatch.setenv("SGPC_MV_STAGE", "0")
    monkeypatch.setenv("SGPC_MV_ROWS", str(rows))
    prob = make_problem("strip", n_e, 3, 2, 0.2, 0.5)
    s = sg.build_system(prob)
    print(f"strip operator n_e={n_e} rows={rows}", flush=True)
    solver = b.SGSolver(prob)
    U = random_block(prob.P, prob.n, seed=n_e)
    Ud = b.to_device_block(U)
    Y = solver.sg_matvec(Ud).cpu().numpy()
    Yo = sg.matvec(s, U.T).T
    assert np.linalg.norm(Y - Yo) <= 1e-12 * np.linalg.norm(Yo)
    for level in (1, 2):
        for direction in (0, 1):
            R = random_block(prob.P, prob.n, seed=level + 10 * direction)
            Rg = solver.sg_coupling(level, direction, b.to_device_block(R), Ud).cpu().numpy()
            lo, hi = s.off[level], s.off[level + 1]
            Ro = R.T.copy()
            if direction == 0:
                Ro[:, :lo] -= sg.level_block(s, slice(0, lo), slice(lo, hi))(U.T[:, lo:hi])
            else:
                Ro[:, lo:hi] -= sg.level_block(s, slice(lo, hi), slice(0, lo))(U.T[:, :lo])
            assert np.linalg.norm(Rg - Ro.T) <= 1e-13 * np.linalg.norm(Ro)
    solver.close()


@pytest.mark.parametrize("rows", [2, 4])
def test_strip_keeps_a_nan_to_its_neighbours(rows, monkeypatch):
    """A NaN at a corner, an edge and an inner node reaches the nodes around it only."""
    from paper_1205_1864_amd import binding as b
    monkeypatch.setenv("SGPC_MV_STAGE", "0")
    monkeypatch.setenv("SGPC_MV_ROWS", str(rows))
    n_e = 65
    nx = n_e - 1
    prob = make_problem("strip", n_e, 2, 1, 0.2, 0.5)
    print(f"strip NaN rows={rows}", flush=True)
    solver = b.SGSolver(prob)
    for iy, ix in ((0, 0), (nx - 1, nx - 1), (0, 31), (32, 0), (33, 31)):
        U = random_block(prob.P, prob.n, seed=1)
        U[0, iy * nx + ix] = np.nan
        Y = solver.sg_matvec(b.to_device_block(U)).cpu().numpy()[0].reshape(nx, nx)
        want = np.zeros((nx, nx), bool)
        want[max(0, iy - 1):iy + 2, max(0, ix - 1):ix + 2] = True
        assert np.array_equal(np.isnan(Y), want)
    solver.close()
