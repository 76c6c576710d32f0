"""The walks of the direct light and of its gradients at the edges of their
launches: receivers that do not fill a wave, lights that do not fill a chunk,
more surfels crossed than one list holds, and a tree deeper than the part of
the walk's stack that lies in LDS."""
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


@pytest.fixture(scope="module")
def orc():
    import oracle as o
    return o


def _sheared(sur):
    """Frames as an optimiser leaves them: neither unit nor orthogonal."""
    s = dict(sur)
    for a in "xyz":
        s["tu" + a] = (sur["tu" + a] * 1.02 + 0.02 * sur["tv" + a]).astype(np.float32)
        s["n" + a] = (sur["n" + a] * 0.97).astype(np.float32)
    return s


@pytest.mark.parametrize("n,lights,sheared", [(1, 3, False), (63, 1, False), (64, 2, True), (65, 5, False), (200, 9, True)])
def test_direct_light_and_gradients_at_wave_edges(g, orc, n, lights, sheared):
    sur = scenes.random_frame_surfels(n, seed=n, scale=(0.1, 0.4))
    if sheared:
        sur = _sheared(sur)
    rng = np.random.default_rng(n)
    lp = (rng.uniform(-0.5, 0.5, (lights, 3)) + [0.0, 0.0, 2.5]).astype(np.float32)
    lI = rng.uniform(1.0, 4.0, lights).astype(np.float32)
    alb = scenes.seeded_array((n, 3), 1, 0.2, 0.9)
    gE = scenes.seeded_array((n, lights, 4, 3), 2, -1.0, 1.0)
    bvh = g.build_bvh(dev_surfels(sur))
    E = g.direct_light(bvh, dev(alb), dev(lp), dev(lI), 4)
    te = orc.default_t_eps(sur)
    assert rel_err(E.cpu().numpy(), orc.direct_light(sur, alb, lp, lI, 4)) < TOL
    got = g.direct_light_backward(bvh, dev(alb), dev(lp), dev(lI), dev(gE))
    want = orc.direct_light_backward(sur, alb, lp, lI, gE, t_eps=te)
    for a, b in zip(got[:3], want[:3]):
        assert rel_err(a.cpu().numpy(), b) < TOL
    for f in orc.GEOMETRY_FIELDS:
        assert rel_err(got[3][f].cpu().numpy(), want[3][f]) < TOL, f


def test_lights_in_one_launch_equal_lights_alone(g):
    """Chunks of lights and the walks' packets do not change a bit of E."""
    sc = scenes.make_config("fruit_bowl", n=3000)
    bvh = g.build_bvh(dev_surfels(sc.surfels))
    lp = np.random.default_rng(1).uniform(-0.4, 0.4, (37, 3)).astype(np.float32) + np.float32([0.0, 1.4, 0.0])
    lI = np.linspace(1.0, 4.0, 37).astype(np.float32)
    E = g.direct_light(bvh, dev(sc.albedo), dev(lp), dev(lI), 4)
    for k in (0, 17, 36):
        one = g.direct_light(bvh, dev(sc.albedo), dev(lp[k:k + 1]), dev(lI[k:k + 1]), 4)
        assert np.array_equal(one.cpu().numpy()[:, 0], E.cpu().numpy()[:, k])


def test_walks_below_the_stack_in_lds(g, orc):
    """A tree of height 34 and more: segment walks push past the entries that
    lie in LDS, packets past 32."""
    from oracle import center
    sur = scenes.deep_chain(copies=4)
    n = sur["px"].shape[0]
    bvh = g.build_bvh(dev_surfels(sur))
    assert bvh.height() >= 32
    alb = np.full((n, 3), 0.5, np.float32)
    lp, lI = np.array([[2.0, 3.0, 9.0]], np.float32), np.array([2.0], np.float32)
    E = g.direct_light(bvh, dev(alb), dev(lp), dev(lI), 1)
    assert rel_err(E.cpu().numpy(), orc.direct_light(sur, alb, lp, lI, 1)) < TOL
    rng = np.random.default_rng(0)
    rows = np.repeat(np.arange(n), 8)
    cols = np.stack([np.sort(rng.choice(np.delete(np.arange(n), i), 8, replace=False)) for i in range(n)]).ravel()
    P = g.ff_from_csr(dev(np.arange(n + 1, dtype=np.int64) * 8), dev(cols.astype(np.int32)),
                      dev(np.ones(cols.size, np.float32)))
    same = np.all([sur["p" + a][rows] == sur["p" + a][cols] for a in "xyz"], axis=0)   # no segment between equal centres
    lam = np.full(n, 0.5, np.float32)
    F = g.ff_center(bvh, P, dev(lam)).csr()[2].cpu().numpy()
    Fo, _ = center.center_ff(sur, rows, cols.astype(np.int32), lam.astype(np.float64), t_eps=orc.default_t_eps(sur))
    assert rel_err(F[~same], Fo[~same]) < TOL
