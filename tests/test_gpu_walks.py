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


@pytest.mark.parametrize("n", [9, 16, 17, 256, 257, 530])
def test_monte_carlo_draws_pick_by_the_running_sum(g, n):
    """One group of n members: each receiver's draw is known from the counter
    generator and the FP64 running sum of the member weights, and its estimate
    from the oracle's centre form factor.  Lists end inside a row of 16 lanes
    and at its edge, and are longer than 16 rows.  Tolerances: an FP32 running
    sum of n terms is off by at most n 2^-24 of the total and its terms by some
    20 roundings, so draws closer than (n + 50) 2^-23 to a step of the sum are
    left out; an estimate has in addition the transmittance's product of at
    most 200 factors, and cosines n . v that lose digits as they near 0."""
    from oracle import center
    from oracle import oracle as orc
    sc = scenes.make_config("box_room", n=n)
    sur, n = sc.surfels, sc.n
    bvh = g.build_bvh(dev_surfels(sur))
    mc = g.mc_create(bvh, groups=1, kmeans_iters=1)
    lam = scenes.seeded_array((n,), seed=5, lo=0.5, hi=1.5).astype(np.float32)
    rho = orc.rho(sur["opacity"], sc.albedo).astype(np.float32)
    E = orc.direct_light(sur, sc.albedo, sc.light_pos, sc.light_I, 1).astype(np.float32)
    B = (E + 0.05 * scenes.seeded_array(E.shape, seed=3, lo=0.5, hi=1.5)).astype(np.float32)
    seed, step = 77, 3
    got = g.mc_estimate(mc, dev(lam), dev(rho), dev(E), dev(B), seed=seed, step=step).cpu().numpy()

    p = np.stack([sur[k] for k in ("px", "py", "pz")], 1).astype(np.float64)
    nrm = np.stack([sur[k] for k in ("nx", "ny", "nz")], 1).astype(np.float64)
    lum = np.maximum(B.astype(np.float64) @ [0.2126, 0.7152, 0.0722], 0).sum((1, 2))
    v = p[None] - p[:, None]
    r2 = (v ** 2).sum(2)
    np.fill_diagonal(r2, 1.0)
    ca, cj = np.abs((nrm[:, None] * v).sum(2)), np.abs((nrm[None] * v).sum(2))
    w = lum[None] * ca * cj / r2 ** 2
    np.fill_diagonal(w, 0.0)
    u = np.empty(n)
    for a in range(n):
        counter = (a | step << 64 | 2 << 192) - 1
        word = np.random.Philox(key=seed, counter=counter).random_raw(2)[1]
        u[a] = (int(word) >> 40) * 2.0 ** -24
    cdf = np.cumsum(w, 1)
    total = cdf[:, -1]
    pick = (cdf <= (u * total)[:, None]).sum(1)
    pick = np.minimum(pick, n - 1)
    gap = np.abs(cdf - (u * total)[:, None]).min(1) / total
    sure = (gap > (n + 50) * 2.0 ** -23) & (u > (n + 50) * 2.0 ** -23)
    assert sure.mean() > 0.9
    rows = np.arange(n)
    F, _ = center.center_ff(sur, rows, pick.astype(np.int32), lam)
    pj = w[rows, pick] / total
    want = E + (rho[:, None, None, :] * (F / pj)[:, None, None, None] * B[pick])
    lost = 8 * np.sqrt(r2[rows, pick]) * (1 / ca[rows, pick] + 1 / cj[rows, pick])
    tol = (n + 250 + lost[:, None, None, None]) * 2.0 ** -23 * np.abs(want - E) + 2.0 ** -23 * np.abs(want)
    bad = np.abs(got - want) > tol
    assert not bad[sure].any(), (np.abs(got - want) / np.abs(want))[sure].max()


def _sheets(before, beyond, layers, seed=0):
    """Surfel 0 looks at `layers` wide thin sheets and at small surfels, some
    before and some beyond them."""
    rng = np.random.default_rng(seed)
    n = 1 + before + beyond + layers
    p = rng.uniform(-0.3, 0.3, (n, 3))
    p[0] = 0.0
    p[1:1 + before, 2] = rng.uniform(0.5, 0.9, before)
    p[1 + before:1 + before + beyond, 2] = rng.uniform(3.5, 4.0, beyond)
    p[1 + before + beyond:, 2] = 1.0 + 0.005 * np.arange(layers)
    nrm = rng.normal(0.0, 0.05, (n, 3)) + [0.0, 0.0, 1.0]
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    tu = np.cross(nrm, [0.0, 1.0, 0.0])
    tu /= np.linalg.norm(tu, axis=1, keepdims=True)
    tv = np.cross(nrm, tu)
    size = np.full(n, 0.01)
    size[1 + before + beyond:] = 0.8
    op = np.full(n, 0.5)
    op[1 + before + beyond:] = 0.01
    cols = {"su": size, "sv": size, "opacity": op}
    for name, v in (("p", p), ("tu", tu), ("tv", tv), ("n", nrm)):
        for k, a in enumerate("xyz"):
            cols[name + a] = v[:, k]
    return {k: np.ascontiguousarray(v, np.float32) for k, v in cols.items()}


@pytest.mark.parametrize("before,beyond,layers", [(1, 0, 1), (0, 33, 3), (500, 12, 40), (300, 213, 40), (0, 600, 150),
                                                  (512, 200, 400)])
def test_center_gradients_of_long_rows_and_lists(g, orc, before, beyond, layers):
    """Rows of one segment, of a chunk and one more, and rows whose crossings
    (90,000 and, in the second chunk, 80,000) do not fit the lists."""
    from oracle import center
    sur = _sheets(before, beyond, layers)
    n, m = sur["px"].shape[0], before + beyond
    bvh = g.build_bvh(dev_surfels(sur))
    ptr = np.full(n + 1, m, np.int64)
    ptr[0] = 0
    cols = np.arange(1, 1 + m, dtype=np.int32)
    P = g.ff_from_csr(dev(ptr), dev(cols), dev(np.ones(m, np.float32)))
    lam = scenes.seeded_array((n,), 7, 0.2, 0.8)
    gF = scenes.seeded_array((m,), 8, -1.0, 1.0)
    F = g.ff_center(bvh, P, dev(lam))
    rows, te = np.zeros(m, np.int64), orc.default_t_eps(sur)
    Fo, _ = center.center_ff(sur, rows, cols, lam.astype(np.float64), t_eps=te)
    assert rel_err(F.csr()[2].cpu().numpy(), Fo) < TOL
    gl, gf = g.ff_center_backward(bvh, F, dev(lam), dev(gF))
    glo, gfo = center.center_backward(sur, rows, cols, lam.astype(np.float64), gF.astype(np.float64), t_eps=te)
    assert rel_err(gl.cpu().numpy(), glo) < TOL
    for f in center.FIELDS:
        assert rel_err(gf[f].cpu().numpy(), gfo[f]) < TOL, f
    again = g.ff_center_backward(bvh, F, dev(lam), dev(gF))
    assert all(torch.equal(gf[f], again[1][f]) for f in gf) and torch.equal(gl, again[0])
