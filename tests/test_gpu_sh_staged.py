"""The directional transfer's sampled products on either side of the rule that
chooses between rows staged in LDS and rows read by their own lanes."""
import numpy as np
import pytest
import scipy.sparse as sp

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, dev_surfels, rel_err  # noqa: E402

TOL = 1e-4   # of the largest value: FP32 sums of at most 130 entries


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


# (rows, mean length 64 or 12): own lanes for K = 1 everywhere but at 30,005
# rows of 64; for K = 4 at 1,024 rows and short ones; for K = 9 also at 2,050 short
@pytest.mark.parametrize("K,Lt,n,short", [(1, 2, 30005, False), (1, 1, 30005, True), (4, 2, 1024, False),
                                          (4, 1, 1025, False), (4, 2, 2048, True), (4, 1, 2050, True),
                                          (9, 2, 1025, False), (9, 1, 2050, True), (16, 1, 1025, True)])
def test_sampled_products_either_way(g, K, Lt, n, short):
    from oracle import sh as osh
    nb = 2
    sur = scenes.random_frame_surfels(n, seed=n)
    lens = np.resize([0, 1, 5, 12, 40] if short else [0, 63, 64, 65, 128], n)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    # every row's senders follow it at a stride: none is its own
    row = np.repeat(np.arange(n), lens)
    cols = (row + 1 + 7 * (np.arange(ptr[-1]) - np.repeat(ptr[:-1], lens))) % n
    order = np.lexsort((cols, row))
    cols = cols[order].astype(np.int32)
    vals = (np.random.default_rng(K).uniform(0.1, 1.0, cols.size) / 130).astype(np.float32)
    F = sp.csr_matrix((vals.astype(np.float64), cols, ptr), shape=(n, n))
    ff = g.ff_from_csr(dev(ptr), dev(cols), dev(vals))
    bvh = g.build_bvh(dev_surfels(sur))
    R = scenes.seeded_array((n, K, 3), 4, 0.1, 0.9)
    E = scenes.seeded_array((n, Lt, K, 3), 5)
    gB = scenes.seeded_array((n, Lt, K, 3), 6, -1, 1)
    B, tape = g.transport_solve_sh(ff, bvh, dev(R), dev(E), nb)
    gE, gR, gF = g.transport_backward_sh(ff, bvh, tape, dev(R), dev(gB))
    Bo, tp = osh.bounce(F, sur, R.astype(np.float64), E, nb, keep_tape=True)
    gEo, gRo, gFo = osh.adjoint(F, sur, R.astype(np.float64), tp, gB)
    for got, want in ((B, Bo), (gE, gEo), (gR, gRo), (gF, gFo)):
        assert rel_err(got.cpu().numpy(), want) < TOL
