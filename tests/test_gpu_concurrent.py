"""Several handles solving at once, each on its own stream and host thread: the blocks
that share a column wait for each other while other launches hold compute units, and
every result is the one of a solve alone, bit for bit."""

import threading

import pytest

pytestmark = pytest.mark.gpu

from sg_inputs import make_problem, named_problem  # noqa: E402


# blocks per column: three (256^2), two (200^2), eleven (513^2); FP32 and a warm start among them
KINDS = [dict(n_e=256, M=5, p=2, prec=64), dict(n_e=200, M=6, p=2, prec=32), dict(n_e=513, M=3, p=1, prec=64, warm=True)]


def test_handles_on_their_own_streams():
    import torch
    from paper_1205_1864_amd import binding as b
    runs = []
    for k in KINDS:
        prob = make_problem("con", k["n_e"], k["M"], k["p"], 0.2, 0.5)
        stream = torch.cuda.Stream()
        solver = b.SGSolver(prob, b.Options(inner_precision=k["prec"], cheb_degree=8, inner_rtol=1e-4,
                                            warm_start=k.get("warm", False)), stream=stream)
        F = b.to_device_block(prob.load_block())
        ref, st = solver.sg_solve(F, rtol=1e-8, maxit=100)
        assert st["rc"] == 0
        torch.cuda.synchronize()
        runs.append((solver, stream, F, ref.clone(), st))
    prob = named_problem("small", L=0.5, n_e=10, M=4, p=4)
    lognormal_stream = torch.cuda.Stream()
    with torch.cuda.stream(lognormal_stream):
        op = b.LognormalOperator(prob, 1.0, 0.5)
    Fl = b.to_device_block(prob.load_block())
    Vref, sl = op.solve(Fl, rtol=1e-8)
    torch.cuda.synchronize()
    out, errors = {}, []

    def solve(i):
        try:
            solver, stream, F, _, _ = runs[i]
            torch.cuda.set_device(0)
            with torch.cuda.stream(stream):
                for _ in range(3):
                    out[i] = solver.sg_solve(F, rtol=1e-8, maxit=100)
        except Exception as exc:  # noqa: BLE001
            errors.append(exc)

    def solve_lognormal():
        try:
            torch.cuda.set_device(0)
            with torch.cuda.stream(lognormal_stream):
                out["logn"] = op.solve(Fl, rtol=1e-8)
        except Exception as exc:  # noqa: BLE001
            errors.append(exc)

    print("concurrent handles", flush=True)
    threads = [threading.Thread(target=solve, args=(i,)) for i in range(len(runs))]
    threads.append(threading.Thread(target=solve_lognormal))
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for i, (solver, _, _, ref, st) in enumerate(runs):
        U, su = out[i]
        assert su["rc"] == 0 and su["outer_it"] == st["outer_it"] and su["inner_it_total"] == st["inner_it_total"]
        assert bool((U == ref).all()), KINDS[i]
        solver.close()
    # a repeat (the device was held for a second) would iterate on the host, to the same tolerance
    V, sv = out["logn"]
    assert sv["rc"] == 0 and sv["outer_it"] == sl["outer_it"]
    assert float((V - Vref).norm()) <= 2e-9 * float(Vref.norm())
    op.close()
