"""The one-launch block solves of the lognormal path at the edges of their shapes:
unknowns per thread, one and several blocks, coefficients held and streamed, and
the systems that stay with the iteration on the host."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import krylov, lognormal, sg  # noqa: E402
from sg_inputs import named_problem  # noqa: E402

# largest block system -> what holds it
CASES = [
    dict(n_e=3, M=2, p=2),    # 3 unknowns: one wave
    dict(n_e=17, M=1, p=1),   # 256: one wave exactly full
    dict(n_e=18, M=1, p=1),   # 289: 512 threads
    dict(n_e=33, M=1, p=2),   # 1024: two per thread exactly
    dict(n_e=65, M=1, p=1),   # 4096: eight per thread exactly
    dict(n_e=10, M=4, p=4),   # 2835 in 35 columns: several lanes per row, held
    dict(n_e=33, M=4, p=2),   # 10240: twenty per thread exactly
    dict(n_e=81, M=2, p=2),   # 19200: thirty-eight per thread, streamed
    dict(n_e=90, M=2, p=2),   # 23763: too many unknowns for the launch
]


# spins = 0: every exchange that has to wait gives up at once, and the solve is
# repeated with its iterations on the host
@pytest.mark.parametrize("spins", [None, "0"])
@pytest.mark.parametrize("pc", ["hsc", "bgs", "mean"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "ne{n_e}-M{M}-p{p}".format(**c))
def test_block_solves_in_one_launch(case, pc, spins, monkeypatch):
    from paper_1205_1864_amd import binding as b
    if spins is not None:
        monkeypatch.setenv("SGPC_LOGN_SPINS", spins)
    prob = named_problem("small", L=0.5, **case)
    print(f"lognormal block solves {case} {pc} spins={spins}", flush=True)
    ls = lognormal.build(prob, 0.5)
    F = prob.load_block()
    res, _ = lognormal.solve_fcg(ls, F.T.copy(), pc, rtol=1e-8)
    op = b.LognormalOperator(prob, 1.0, 0.5)
    U, st = op.solve(b.to_device_block(F), rtol=1e-8, precond=pc)
    assert st["rc"] == 0
    # block solves to 1e-12 leave the count and the solution of exact ones
    assert st["outer_it"] == res.iterations
    Ug = U.cpu().numpy()
    assert np.linalg.norm(Ug - res.x.T) <= 1e-9 * np.linalg.norm(res.x)
    r = sg.vec(F.T) - ls.A @ sg.vec(Ug.T)
    assert np.linalg.norm(r) <= 1.01e-8 * np.linalg.norm(F)
    op.close()
