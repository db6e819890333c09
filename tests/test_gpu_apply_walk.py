"""eik_apply_local walks planes: grids large enough for walks of several planes
with a remainder, barriers, unreached neighbours and both local solves, bit for
bit against the oracle."""

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
eik = pytest.importorskip("paper_2106_15869_amd")

pytestmark = pytest.mark.gpu


# n >> 19 planes per walk: 2 (odd number of planes), 4 (remainder 1 and 3), 1
@pytest.mark.parametrize("shape", [(1027, 1025), (17, 300, 257), (33, 200, 330), (1023, 2100), (2, 3, 5), (1, 1)])
@pytest.mark.parametrize("h", [0.7, 0.7 * 2.0 ** -60])
def test_walks_bitwise(shape, h):
    rng = np.random.default_rng(3)
    F = rng.uniform(0.2, 3.0, size=shape).astype(np.float32)
    F[rng.random(shape) < 0.05] = 0.0
    phi = (h * rng.uniform(0.0, 4.0, size=shape)).astype(np.float32)
    phi[rng.random(shape) < 0.3] = np.inf
    print(f"[case] apply_local {shape} h {h}", flush=True)
    got = eik.apply_local(torch.from_numpy(F).cuda(), torch.from_numpy(phi).cuda(), h).cpu().numpy()
    want = oracle.apply_local(F, h, phi, dtype=np.float32)
    np.testing.assert_array_equal(got, want)
