"""Tiles that hold nodes for both local solves of a visit: ordinary speeds and
a few whose H = h / F lies outside the short solve's range, so that the waves
of a workgroup differ in what their nodes need.  Every value is a fixed point
of the exact local solve on its neighbours' values, and exactly the nodes that
can be reached are finite."""

import numpy as np
import pytest

import oracle
from tests import helpers as H

torch = pytest.importorskip("torch")
eik = pytest.importorskip("paper_2106_15869_amd")

pytestmark = pytest.mark.gpu

# 2^k: speeds outside the short solve's range on either side (equal spacing:
# H in 2^-30 .. 2^50 for float32, 2^-400 .. 2^400 for float64; per axis
# 2^-30 .. 2^30 and 2^-200 .. 2^200)
FAST = {("float32", False): 40, ("float64", False): 420, ("float32", True): 40, ("float64", True): 220}
SLOW = {("float32", False): -55, ("float64", False): -420, ("float32", True): -36, ("float64", True): -220}


def field(dims, dtype, aniso, share, seed):
    r = np.random.default_rng(seed)
    F = r.uniform(0.2, 3.0, size=dims)
    u = r.random(dims)
    F[u < share] = 2.0 ** FAST[(dtype, aniso)]
    F[u > 1 - share] = 2.0 ** SLOW[(dtype, aniso)]
    F[r.random(dims) < 0.05] = 0.0
    F.reshape(-1)[0] = 1.0
    return F.astype(dtype)


@pytest.mark.parametrize("dims,tile,aniso", [
    ((37, 50), None, False), ((64, 64), (32, 32), False), ((37, 130), (16, 64), False), ((37, 50), (8, 32), False),
    ((130, 70), (64, 64), False), ((37, 50), None, True),
    ((19, 13, 21), None, False), ((19, 13, 21), (4, 8, 8), False), ((19, 13, 21), (4, 4, 16), False),
    ((19, 13, 21), (8, 8, 16), False), ((19, 33, 21), (16, 16, 16), False), ((19, 13, 21), None, True),
])
@pytest.mark.parametrize("share", [0.002, 0.05])  # a wave or two of a workgroup; most of them
@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_waves_with_both_kinds_of_nodes(dims, tile, aniso, share, dtype):
    sp = ((0.25, 0.4) if len(dims) == 2 else (0.25, 0.4, 0.3)) if aniso else None
    F = field(dims, dtype, aniso, share, 5)
    print(f"[case] mixed {dims} tile {tile} aniso {aniso} share {share} {dtype}", flush=True)
    phi = eik.solve(torch.from_numpy(F).cuda(), 0.25, np.array([0]), tile=tile, spacing=sp).cpu().numpy()
    fin = np.isfinite(phi)
    assert np.array_equal(~fin, H.unreachable_mask(F, [0]))
    m = fin & (F > 0)
    m.flat[0] = False
    G = oracle.apply_local(F.astype(np.float64), 0.25, phi.astype(np.float64), spacing=sp)
    # a local solve is some ten operations on numbers no larger than its result
    # (the sources' value is 0), each rounded to half a unit in the last place
    ulp = np.spacing(np.abs(phi[m])).astype(np.float64)
    assert np.max(np.abs(phi[m].astype(np.float64) - G[m]) / ulp) <= 16
