"""Direct light of small scenes with many lights, a lane to a shadow ray: the
bits of 16 lanes to a ray, which the same lights take a few at a time."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, dev_surfels  # noqa: E402


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


def _scene(n):
    if n == "deep":   # walks past the stack's part in LDS
        return scenes.deep_chain(copies=4)
    return scenes.random_frame_surfels(n, seed=n, scale=(0.1, 0.4))


# either side of 850 lights, of 250,000 rays of 256 lights and more, and of
# 140,000 rays, workgroups that are not full, and one surfel
@pytest.mark.parametrize("n,lights", [(1, 850), (2, 851), (63, 849), (63, 850), (160, 874), (160, 876), (977, 255),
                                      (977, 256), (976, 256), ("deep", 900), ("deep", 2600)])
def test_many_lights_equal_few(g, n, lights):
    sur = _scene(n)
    n = sur["px"].shape[0]
    rng = np.random.default_rng(n)
    lp = dev((rng.uniform(-0.5, 0.5, (lights, 3)) + [0.0, 0.0, 2.5]).astype(np.float32))
    lI = dev(rng.uniform(1.0, 4.0, lights).astype(np.float32))
    alb = dev(scenes.seeded_array((n, 3), 1, 0.2, 0.9))
    bvh = g.build_bvh(dev_surfels(sur))
    parts = [slice(k, min(k + 200, lights)) for k in range(0, lights, 200)]
    E = g.direct_light(bvh, alb, lp, lI, 4)
    assert torch.equal(E, torch.cat([g.direct_light(bvh, alb, lp[s], lI[s], 4) for s in parts], 1))
    assert E.abs().max() > 0
    for K in (1, 4, 9, 16):
        R = dev(scenes.seeded_array((n, K, 3), 2, 0.2, 0.9))
        E = g.direct_light_sh(bvh, R, lp, lI)
        assert torch.equal(E, torch.cat([g.direct_light_sh(bvh, R, lp[s], lI[s]) for s in parts], 1))
