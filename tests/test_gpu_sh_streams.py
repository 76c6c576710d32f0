"""Directional transfer by several streams on one BVH: a solve only reads it."""
import pytest

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, dev_surfels  # noqa: E402


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


def test_solves_on_two_streams_share_a_bvh(g):
    n, K = 3000, 9
    sc = scenes.make_config("fruit_bowl", n=n)
    bvh = g.build_bvh(dev_surfels(sc.surfels))
    ffs = [g.form_factors(bvh, 64, s, t_min=1e-4) for s in (1, 2)]
    R = dev(scenes.seeded_array((n, K, 3), 4, 0.1, 0.9))
    E = dev(scenes.seeded_array((n, 1, K, 3), 5))
    gB = dev(scenes.seeded_array((n, 1, K, 3), 6, -1.0, 1.0))

    def both(ff):
        B, tape = g.transport_solve_sh(ff, bvh, R, E, 4)
        return (B, *g.transport_backward_sh(ff, bvh, tape, R, gB))

    want = [both(ff) for ff in ffs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = [[], []]
    for _ in range(5):
        for k, (st, ff) in enumerate(zip(streams, ffs)):
            with torch.cuda.stream(st):
                got[k].append(both(ff))
    torch.cuda.synchronize()
    for k in range(2):
        for out in got[k]:
            assert all(torch.equal(a, b) for a, b in zip(out, want[k]))
