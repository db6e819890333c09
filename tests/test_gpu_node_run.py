"""Deterministic node lists: short lists run many iterations in one launch,
longer ones two launches each.  Grids whose lists are short throughout, cross
the limit (2048 nodes) in STEP 2 or in the remedy, or are too large for the
short form give the serial emulation's values and counts exactly."""

import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
eik = pytest.importorskip("paper_2106_15869_amd")

pytestmark = pytest.mark.gpu

KEYS = ("step2_iters", "step3_iters", "evals_step2", "evals_detect", "evals_remedy", "remedy_initial", "max_active")


@pytest.mark.parametrize("P,crosses", [
    (W.lognormal_2d(24, seed=1), False),          # every list short
    (W.lognormal_2d(160, seed=2), True),          # the remedy's lists cross the limit
    (W.layered_3d(46), True),                     # so does the front (a face of 46^2 nodes)
    (W.maze_3d(30, seed=5), True),
    (W.layered_3d(50), True),                     # too many nodes for the short form
], ids=lambda v: getattr(v, "name", str(v)))
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_short_and_long_lists_match_emulation(P, crosses, dtype):
    F = torch.from_numpy(P.F.astype(dtype)).cuda()
    print(f"[case] {P.name} {np.dtype(dtype).name}", flush=True)
    phi, st = eik.solve(F, P.h, P.sources, variant="node", deterministic=True, stats=True)
    want, wst = oracle.ifim(P.F.astype(dtype), P.h, P.sources, dtype=dtype)
    assert np.array_equal(phi.cpu().numpy(), want)
    for k in KEYS:
        assert st[k] == wst[k], (k, st[k], wst[k])
    longest = max(st["max_active"], st["evals_remedy"] // max(st["step3_iters"], 1), st["remedy_initial"])
    assert (longest > 2048) == crosses, longest
