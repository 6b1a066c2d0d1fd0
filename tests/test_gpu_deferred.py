"""Loop reductions completed by the passes that need them against launches of their own (FGH_DEFER=0): the
same partial sums, added in the same order, give the same scalars, so iterates, counts and test
quantities are bitwise equal.  CG (beta in the first pass, alpha in the pass after it or in the
update kernel) and the other solvers, on specialised, run-time-length and mixed-radix passes, in 2D
and 3D, both precisions and rules; loops that end on the tolerance, on a fixed count and on
max_iter; batches."""
import numpy as np
import pytest

from paper_1508_02045_amd import inputs as I
from test_gpu_batch import batch, members

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FP64, REFINED = 0, 1
# 135 x 135 x 45: more partial sums than a workgroup adds up for itself (the end is a launch, alpha is not)
GRIDS = [((63, 81), 0, FP64), ((63, 81), 0, REFINED), ((45, 63, 81), 0, FP64), ((45, 63, 81), 0, REFINED),
         ((51, 85), 0, FP64), ((51, 85), 0, REFINED), ((17, 15, 19), 0, FP64), ((17, 15, 19), 0, REFINED),
         ((21, 15, 27), 0, REFINED), ((41, 23), 1, FP64), ((23, 19), 1, REFINED), ((11, 9, 13), 1, FP64),
         ((135, 135, 45), 0, FP64)]


def plan_of(N, rule, prec):
    from paper_1508_02045_amd import fgh
    rng = np.random.default_rng(sum(N) + 3)
    ph = (rng.random(N) < 0.3).astype(np.uint8)
    tab = I.sym_pack(I.iso_tables(len(N), [1.0, 30.0])).T
    return fgh.Plan(N, rule=rule, precision=prec, phase=torch.from_numpy(ph).cuda(), phase_table=tab)


def both(monkeypatch, run):
    """run() with the reductions deferred and in launches of their own: (field, counts and residuals)."""
    out = []
    for on in ("1", "0"):
        monkeypatch.setenv("FGH_DEFER", on)
        e, st, stats = run()
        s = stats[0]
        out.append((e.cpu().numpy(), st, [s[k] for k in ("iters", "outer_iters", "status", "rel_res_recursive")]))
    (e1, st1, s1), (e0, st0, s0) = out
    assert st1 == st0 and s1 == s0, (s1, s0)
    assert np.array_equal(e1, e0)
    return st1, s1


@pytest.mark.parametrize("solver", ["cg", "richardson", "chebyshev", "eyre_milton"])
@pytest.mark.parametrize("N,rule,prec", GRIDS)
def test_deferred_equals_separate(monkeypatch, N, rule, prec, solver):
    from paper_1508_02045_amd import fgh
    if solver == "eyre_milton" and rule == 1:
        pytest.skip("Eyre-Milton has no exact-integration form")
    d = len(N)
    E = np.array([1.0, -0.5, 0.25][:d])
    plan = plan_of(N, rule, prec)
    print(N, rule, prec, solver, flush=True)
    st, s = both(monkeypatch, lambda: plan.solve(solver, E, 1e-8, max_iter=20000))
    assert st == fgh.FGH_OK
    # the loop ends on max_iter, in the middle of a graph's bodies and of a chunk (refined: each inner loop)
    st, s = both(monkeypatch, lambda: plan.solve(solver, E, 1e-8, max_iter=11))
    assert st == fgh.FGH_E_NO_CONVERGENCE or prec == REFINED
    if prec == FP64:  # fixed-count solves are FP64 only
        for n in (1, 8, 13):
            st, s = both(monkeypatch, lambda: plan.solve_fixed(solver, E, n))
            assert st == fgh.FGH_OK and s[0] == n
    plan.close()


@pytest.mark.parametrize("N,solver", [((81, 81), "cg"), ((45, 45, 45), "cg"), ((81, 81), "eyre_milton")])
def test_batch_deferred_equals_separate(monkeypatch, N, solver):
    ms = members(N, 0, 3, 1, 40 + sum(N))
    out = []
    for on in ("1", "0"):
        monkeypatch.setenv("FGH_DEFER", on)
        st, es, stats, _ = batch(ms, solver)
        assert st == 0
        out.append((es, [(s["iters"], s["outer_iters"], s["rel_res_recursive"]) for s in stats]))
    assert out[0][1] == out[1][1]
    for a, b in zip(out[0][0], out[1][0]):
        assert np.array_equal(a, b)
    for mb in ms:
        mb["plan"].close()
