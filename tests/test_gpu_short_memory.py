"""Gradient calls whose lists do not fit what device memory is free: they take
less, or none, and give the same bits."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, dev_surfels  # noqa: E402

MB = 1 << 20


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


def _leave(size):
    """Takes all device memory but about `size` bytes."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    for _ in range(8):
        more = torch.cuda.mem_get_info()[0] - size
        if more < 16 * MB:
            break
        held.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
    assert torch.cuda.mem_get_info()[0] < size + 32 * MB
    return held


@pytest.mark.parametrize("n,lights,left", [(4096, 512, 400 * MB), (262144, 1, 600 * MB)])
def test_light_gradients(g, n, lights, left):
    """663 MB of lists where 50 MB may be taken (a few lights at a time), and
    83 MB for the one light where 75 MB may (none)."""
    sc = scenes.make_config("fruit_bowl", n=n)
    sur = dev_surfels(sc.surfels)
    rng = np.random.default_rng(0)
    lp = (rng.uniform(-0.4, 0.4, (lights, 3)) + [0.0, 1.4, 0.0]).astype(np.float32)
    args = (dev(sc.albedo), dev(lp), torch.full((lights,), 2.0, device="cuda"),
            dev(scenes.seeded_array((n, lights, 1, 3), 2, -1.0, 1.0)))
    bvh = g.build_bvh(sur)
    want = g.direct_light_backward(bvh, *args)
    del bvh
    bvh = g.build_bvh(sur)
    torch.cuda.synchronize()
    full = _leave(left)
    try:
        for _ in range(2):
            got = g.direct_light_backward(bvh, *args)
            assert all(torch.equal(a, b) for a, b in zip(got[:3], want[:3]))
            assert all(torch.equal(got[3][f], want[3][f]) for f in want[3])
    finally:
        del full
        torch.cuda.empty_cache()


def test_center_gradients(g):
    """273 MB of lists where 19 MB may be taken."""
    n = 2000
    sc = scenes.make_config("fruit_bowl", n=n)
    bvh = g.build_bvh(dev_surfels(sc.surfels))
    P = g.form_factors(bvh, 64, 3, t_min=1e-4)
    lam = dev(scenes.seeded_array((n,), 7, 0.2, 0.8))
    gF = dev(scenes.seeded_array((P.info()[1],), 8, -1.0, 1.0))
    F = g.ff_center(bvh, P, lam)
    want = g.ff_center_backward(bvh, F, lam, gF)
    F = g.ff_center(bvh, P, lam)
    full = _leave(150 * MB)
    try:
        for _ in range(2):
            got = g.ff_center_backward(bvh, F, lam, gF)
            assert torch.equal(got[0], want[0])
            assert all(torch.equal(got[1][f], want[1][f]) for f in want[1])
    finally:
        del full
        torch.cuda.empty_cache()


def test_geometry_gradients_of_many_blocks(g):
    """2.2 GB of lists (1,024 blocks of surfels) where 190 MB may be taken: all
    contributions are added directly, and listed once there is room."""
    n = 262145
    bvh = g.build_bvh(dev_surfels(scenes.make_config("fruit_bowl", n=n).surfels))
    ff = g.form_factors(bvh, 16, 3, t_min=1e-4, topk=64)
    gF = dev(scenes.seeded_array((ff.info()[1],), 8, -1.0, 1.0))
    full = _leave(1500 * MB)
    try:
        direct = g.geometry_backward(bvh, ff, gF)
    finally:
        del full
        torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    listed = g.geometry_backward(bvh, ff, gF)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] > 2000 * MB
    assert all(torch.equal(direct[f], listed[f]) for f in direct)
