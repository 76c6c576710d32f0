"""Batches whose callers move their buffers, and whose scenes are many and
small or of mixed widths, against the scenes one by one."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev  # noqa: E402


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


def _batch(g, sizes, lengths, lights, K):
    ffs = [g.ff_from_csr(*(dev(a) for a in scenes.seeded_csr(n, k, seed=s)))
           for s, (n, k) in enumerate(zip(sizes, lengths))]
    rho = [dev(scenes.seeded_array((n, 3), s, 0.2, 0.9)) for s, n in enumerate(sizes)]
    E = [dev(scenes.seeded_array((n, lt, K, 3), 10 + s)) for s, (n, lt) in enumerate(zip(sizes, lights))]
    return ffs, rho, E, g.batch_create(ffs, lights, K)


def _compare(g, ffs, rho, E, batch, nb, gB, B, out):
    """Bit for bit what every scene gives by itself."""
    gE, gr, gF = out
    B, gE, gB = batch.unpack(B), batch.unpack(gE), batch.unpack(gB)
    r0 = e0 = 0
    for ff, r, e, b, ge, gb in zip(ffs, rho, E, B, gE, gB):
        n, nnz = ff.info()
        Bs, tape = g.transport_solve(ff, r, e, nb)
        gEs, grs, gFs = g.transport_backward(ff, tape, r, gb.contiguous())
        assert torch.equal(b, Bs) and torch.equal(ge, gEs)
        assert torch.equal(gr[r0:r0 + n], grs) and torch.equal(gF[e0:e0 + nnz], gFs)
        r0, e0 = r0 + n, e0 + nnz


def test_adjoint_follows_a_grad_B_that_moves(g):
    sizes, K, nb = [130, 64, 301], 9, 3
    ffs, rho, E, batch = _batch(g, sizes, [40, 10, 90], [1, 3, 2], K)
    flat, rows = batch.pack(E), torch.cat(rho)
    B, gE = g.batch_transport_solve(batch, rows, flat, nb), torch.empty_like(flat)
    held = []
    for s in range(3):
        gB = dev(scenes.seeded_array(tuple(flat.shape), 30 + s, -1.0, 1.0))
        held.append(gB)   # each at an address of its own
        out = g.batch_transport_backward(batch, rows, gB, out=gE)
        _compare(g, ffs, rho, E, batch, nb, gB, B, out)


@pytest.mark.parametrize("K,nb", [(1, 3), (4, 9), (9, 2)])
def test_many_small_scenes(g, K, nb):
    """Scenes of one to 13 chunks, of rows that 16 and 64 lanes take, of one
    surfel and of none but empty rows, and one too large to share launches."""
    sizes = [1, 2, 63, 64, 65, 130, 257, 300, 511, 40, 33000, 90, 200, 129]
    lengths = [0, 1, 5, 30, 60, 12, 40, 100, 20, 0, 10, 70, 150, 9]
    lights = [1, 3, 1, 2, 4, 5, 17, 1, 6, 1, 1, 23, 9, 50]
    ffs, rho, E, batch = _batch(g, sizes, lengths, lights, K)
    flat, rows = batch.pack(E), torch.cat(rho)
    gB = dev(scenes.seeded_array(tuple(flat.shape), 30, -1.0, 1.0))
    B = g.batch_transport_solve(batch, rows, flat, nb)
    _compare(g, ffs, rho, E, batch, nb, gB, B, g.batch_transport_backward(batch, rows, gB))
    # the same layout refilled with rows of other lengths: captured loops, other groups
    other = [g.ff_from_csr(*(dev(a) for a in scenes.seeded_csr(n, k, seed=50 + s)))
             for s, (n, k) in enumerate(zip(sizes, lengths[::-1]))]
    batch = g.batch_create(other, lights, K, batch=batch)
    B = g.batch_transport_solve(batch, rows, flat, nb)
    _compare(g, other, rho, E, batch, nb, gB, B, g.batch_transport_backward(batch, rows, gB))
