"""Synchronous tile solves with an explicit launch budget.  The correcting
update step does the work of the update step alone and of the remedy loop, so
a budget of half the launches it takes (each of the two loops fitted into
that) has to converge: what the update step leaves over goes to the remedy
loop.  Budgets far too short are still reported."""

import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
eik = pytest.importorskip("paper_2106_15869_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _problems():
    r = np.random.default_rng(3)
    return [W.lognormal_2d(300, seed=4), W.maze_3d(40, seed=3), W.paper_example(1, 300),
            W.Problem("strip_1x700", np.exp(r.normal(size=(1, 700))).astype(np.float32), 0.5, np.array([0]))]


@pytest.mark.parametrize("call", ["solve", "fifo", "noalloc", "batch"])
@pytest.mark.parametrize("part", [2, 3])  # budget: the launches without one over this
@pytest.mark.parametrize("P", _problems(), ids=lambda P: P.name)
def test_remedy_takes_up_what_the_update_budget_left(P, part, call):
    F = torch.from_numpy(P.F).to(DEV)
    fifo = call == "fifo"

    def run(budget):
        if call == "noalloc":
            return eik.solve_noalloc(F, P.h, P.sources, source_values=P.source_values, max_iters=budget, stats=True)
        if call == "batch":
            vals = None if P.source_values is None else [P.source_values]
            phi, st = eik.solve_batch(F.reshape(-1), [P.F.shape], P.h, [P.sources], source_values=vals,
                                      max_iters=budget, stats=True)
            return phi.view(P.F.shape), st
        return eik.solve(F, P.h, P.sources, source_values=P.source_values, fifo=fifo, max_iters=budget, stats=True)

    _, st = run(0)
    n = st["step2_iters"] + st["step3_iters"]
    # a few to spare: visits race, so the number of launches differs from run to run
    budget = -(-n // part) + 4
    print(f"[case] {P.name} {call}: {n} launches, budget {budget}", flush=True)
    got, st = run(budget)
    ref = oracle.fmm(P.F.astype(np.float64), P.h, P.sources, values=P.source_values)
    assert np.max(np.abs(got.cpu().numpy() - ref)) <= 1e-5 * ref.max()
    with pytest.raises(eik.EikError) as e:
        run(max(1, n // 8))
    assert e.value.status == eik.EIK_ERR_NO_CONVERGENCE
