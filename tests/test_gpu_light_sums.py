"""Direct-light gradients whose segments cross more surfels than the lists have
room for, and whose lights take more than one slice of the lists."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, dev_surfels, rel_err  # noqa: E402

TOL = 1e-4   # of the largest value: FP32 terms, 64-bit fixed-point sums


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


def _stack(layers, per_layer, seed=0):
    """Wide thin sheets above each other, all facing the light: a sheet's
    shadow segment crosses those of every layer above it."""
    rng = np.random.default_rng(seed)
    n = layers * per_layer
    p = rng.uniform(-0.05, 0.05, (n, 3))
    p[:, 2] = 0.02 * (np.arange(n) // per_layer) + rng.uniform(0.0, 0.004, n)
    nrm = rng.normal(0.0, 0.03, (n, 3)) + [0.0, 0.0, 1.0]
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    tu = np.cross(nrm, [0.0, 1.0, 0.0])
    tu /= np.linalg.norm(tu, axis=1, keepdims=True)
    tv = np.cross(nrm, tu)
    cols = {"su": np.full(n, 0.9), "sv": np.full(n, 0.9), "opacity": np.full(n, 0.02)}
    for name, v in (("p", p), ("tu", tu), ("tv", tv), ("n", nrm)):
        for k, a in enumerate("xyz"):
            cols[name + a] = v[:, k]
    return {k: np.ascontiguousarray(v, np.float32) for k, v in cols.items()}


@pytest.mark.parametrize("layers,per_layer", [(70, 12), (110, 24)])
def test_more_long_segments_than_blocks(g, orc, layers, per_layer):
    """Of 840 (2,640) sheets in 70 (110) layers far more than one in eight
    cross over 64 others, in the second scene many over 160 too: whichever
    segments the blocks go to, the gradients are the same bits."""
    sur = _stack(layers, per_layer)
    n = sur["px"].shape[0]
    alb = scenes.seeded_array((n, 3), 1, 0.2, 0.9)
    gE = scenes.seeded_array((n, 1, 1, 3), 2, -1.0, 1.0)
    lp, lI = np.array([[0.1, -0.2, 6.0]], np.float32), np.array([3.0], np.float32)
    bvh = g.build_bvh(dev_surfels(sur))
    args = (bvh, dev(alb), dev(lp), dev(lI), dev(gE))
    got = g.direct_light_backward(*args)
    want = orc.direct_light_backward(sur, alb, lp, lI, gE, t_eps=orc.default_t_eps(sur))
    for a, b in zip(got[:3], want[:3]):
        assert rel_err(a.cpu().numpy(), b) < TOL
    for f in orc.GEOMETRY_FIELDS:
        assert rel_err(got[3][f].cpu().numpy(), want[3][f]) < TOL, f
    for _ in range(20):
        again = g.direct_light_backward(*args)
        assert all(torch.equal(a, b) for a, b in zip(got[:3], again[:3]))
        assert all(torch.equal(got[3][f], again[3][f]) for f in orc.GEOMETRY_FIELDS)


def test_more_lights_than_one_slice(g, orc):
    """63 surfels are padded to 256 places a light, so 8,192 lights fill the
    lists: eight more are a slice of their own, the albedo's sum goes on from
    the first, and both are walked again between the passes."""
    sur = scenes.random_frame_surfels(63, seed=4, scale=(0.1, 0.4))
    lights = 8200
    rng = np.random.default_rng(5)
    lp = (rng.uniform(-0.5, 0.5, (lights, 3)) + [0.0, 0.0, 2.5]).astype(np.float32)
    lI = rng.uniform(1.0, 4.0, lights).astype(np.float32)
    alb = scenes.seeded_array((63, 3), 1, 0.2, 0.9)
    gE = scenes.seeded_array((63, lights, 1, 3), 2, -1.0, 1.0)
    bvh = g.build_bvh(dev_surfels(sur))
    args = (bvh, dev(alb), dev(lp), dev(lI), dev(gE))
    got = g.direct_light_backward(*args)
    want = orc.direct_light_backward(sur, alb, lp, lI, gE, t_eps=orc.default_t_eps(sur))
    for a, b in zip(got[:3], want[:3]):
        assert rel_err(a.cpu().numpy(), b) < TOL
    for f in orc.GEOMETRY_FIELDS:
        assert rel_err(got[3][f].cpu().numpy(), want[3][f]) < TOL, f
    again = g.direct_light_backward(*args)
    assert all(torch.equal(a, b) for a, b in zip(got[:3], again[:3]))
    assert all(torch.equal(got[3][f], again[3][f]) for f in orc.GEOMETRY_FIELDS)
