"""eik_apply_local on narrow planes, whose lanes run through several walks: bit
for bit against the oracle."""

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
eik = pytest.importorskip("paper_2106_15869_amd")

pytestmark = pytest.mark.gpu


def case(shape, dtype, seed=4, h=0.7):
    rng = np.random.default_rng(seed)
    F = rng.uniform(0.2, 3.0, size=shape).astype(dtype)
    F[rng.random(shape) < 0.05] = 0.0
    phi = (h * rng.uniform(0.0, 4.0, size=shape)).astype(dtype)
    phi[rng.random(shape) < 0.3] = np.inf
    return F, phi, h


# one, two (fewer than 16 nodes a plane), three and eight planes a walk, with remainders
@pytest.mark.parametrize("shape", [(5, 1), (1100001, 1), (300001, 7), (40001, 15), (98303, 16), (260001, 17), (4097, 257),
                                   (70001, 4, 4), (1, 3, 5), (70001, 1, 16), (2001, 63, 33), (3, 1, 1)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_narrow_planes_bitwise(shape, dtype):
    F, phi, h = case(shape, dtype)
    print(f"[case] apply_local {shape} {np.dtype(dtype).name}", flush=True)
    got = eik.apply_local(torch.from_numpy(F).cuda(), torch.from_numpy(phi).cuda(), h).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.apply_local(F, h, phi, dtype=dtype))
