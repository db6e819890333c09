"""eik_tune times a configuration once: the zero tile is the default shape."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
eik = pytest.importorskip("paper_2106_15869_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(23, 41), (11, 9, 13)])  # size classes no other test tunes
def test_no_shape_twice(shape):
    F = torch.from_numpy(np.random.default_rng(1).uniform(0.5, 2.0, size=shape)).cuda()
    print(f"[case] tune {shape}", flush=True)
    cands = eik.tune(F, 0.5, np.array([0]))["candidates"]
    default = (1, 16, 16) if len(shape) == 2 else (8, 8, 8)
    seen = [(c["tile"] if any(c["tile"]) else default, c["inner_iters"], c["order_min"], c["workgroups"]) for c in cands]
    assert len(seen) == len(set(seen)), seen
