"""The directional transfer's staged rows at their edges: rows of a batch of
64 entries and of one more or less, empty rows, each number of coefficients,
light blocks that are not a multiple of 16 bytes from the buffer's start."""
import numpy as np
import pytest
import scipy.sparse as sp

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, dev_surfels, rel_err  # noqa: E402

TOL = 1e-4   # of the largest value: FP32 sums of at most 200 entries


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("K,Lt", [(1, 1), (1, 3), (4, 1), (4, 2), (9, 1), (9, 2), (16, 1), (16, 2)])
def test_transfer_at_batch_edges(g, K, Lt, shift):
    from oracle import sh as osh
    sc = scenes.make_config("fruit_bowl", n=210)
    n, nb = sc.n, 3
    rng = np.random.default_rng(K + Lt)
    lens = np.array([0, 1, 63, 64, 65, 127, 128, 129, 191, 193, 200])[np.arange(n) % 11]
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    # no surfel is its own sender: the pair has no direction, and the adjoint
    # takes the normal for it on either side
    cols = np.concatenate([np.sort(rng.choice(np.delete(np.arange(n), i), k, replace=False))
                           for i, k in enumerate(lens)]).astype(np.int32)
    vals = (rng.uniform(0.1, 1.0, cols.size) / 200).astype(np.float32)
    F = sp.csr_matrix((vals.astype(np.float64), cols, ptr), shape=(n, n))
    ff = g.ff_from_csr(dev(ptr), dev(cols), dev(vals))
    bvh = g.build_bvh(dev_surfels(sc.surfels))
    R = scenes.seeded_array((n, K, 3), 4, 0.1, 0.9)
    E = scenes.seeded_array((n, Lt, K, 3), 5)
    gB = scenes.seeded_array((n, Lt, K, 3), 6, -1, 1)

    def at(x):   # x, `shift` floats into a buffer
        flat = torch.empty(x.size + 4, dtype=torch.float32, device="cuda")
        out = flat[shift:shift + x.size].view(x.shape)
        out.copy_(dev(x))
        return out

    B, tape = g.transport_solve_sh(ff, bvh, dev(R), at(E), nb)
    gE, gR, gF = g.transport_backward_sh(ff, bvh, tape, dev(R), at(gB))
    alone, _ = g.transport_solve_sh(ff, bvh, dev(R), at(E), nb, keep_tape=False, out=at(np.zeros_like(E)))
    Bo, tp = osh.bounce(F, sc.surfels, R.astype(np.float64), E, nb, keep_tape=True)
    gEo, gRo, gFo = osh.adjoint(F, sc.surfels, R.astype(np.float64), tp, gB)
    assert torch.equal(B, alone)
    for got, want in ((B, Bo), (gE, gEo), (gR, gRo), (gF, gFo)):
        assert rel_err(got.cpu().numpy(), want) < TOL
