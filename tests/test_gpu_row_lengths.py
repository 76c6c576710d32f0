"""The FP32 row products where rows are short, which 16 or 32 lanes take each
or chunks of columns side by side: lengths around a reading of 16 and of eight
entries, one to thirteen chunks, fewer and more rows than fill the chip."""
import numpy as np
import pytest
import scipy.sparse as sp

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, rel_err  # noqa: E402

# FP32 sums of up to 130 products of values in [0, 1]: 130 x 2^-24 of the
# largest sum bounds one product's error, nine bounces carry nine of them
TOL = 9 * 130 * 2.0 ** -24

LENGTHS = {"few": [0, 1, 2, 7, 8, 9, 15, 16, 17, 33], "some": [0, 1, 16, 31, 32, 33, 48, 49, 64, 65, 100],
           "many": [130, 127, 128, 129, 0, 64]}


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


def _operator(n, lengths, seed):
    """Rows of the given lengths in turn, columns spread over all senders."""
    rng = np.random.default_rng(seed)
    lens = np.resize(lengths, n)
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(lens)
    within = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
    step = np.repeat(np.maximum(1, (n - 1) // np.maximum(lens, 1)), lens)
    col = within * step + np.repeat(rng.integers(0, np.maximum(1, (n - 1) // np.maximum(lens, 1))), lens)
    val = (rng.uniform(0.1, 1.0, col.size) * np.repeat(0.6 / np.maximum(lens, 1), lens)).astype(np.float32)
    return rp, col.astype(np.int32), val


@pytest.mark.parametrize("lights,K", [(1, 1), (1, 4), (1, 9), (17, 1), (2, 16), (3, 16), (10, 9), (49, 4)])
@pytest.mark.parametrize("n,kind,nb", [(230, "few", 9), (230, "some", 2), (8200, "few", 2), (8200, "some", 9),
                                       (8200, "many", 1)])
def test_short_rows(g, orc, lights, K, n, kind, nb):
    if n * lights * K * nb > 8e6:
        nb = 2
    rp, col, val = _operator(n, LENGTHS[kind], seed=lights + K)
    F = sp.csr_matrix((val.astype(np.float64), col, rp), shape=(n, n))
    rho = scenes.seeded_array((n, 3), 1, 0.2, 0.9)
    E = scenes.seeded_array((n, lights, K, 3), 2)
    gB = scenes.seeded_array((n, lights, K, 3), 3)
    ff = g.ff_from_csr(dev(rp), dev(col), dev(val))
    B, tape = g.transport_solve(ff, dev(rho), dev(E), nb)
    gE, grho, gF = g.transport_backward(ff, tape, dev(rho), dev(gB))
    Bo, to = orc.bounce(F, rho, E, nb, keep_tape=True)
    gEo, grhoo, gFo = orc.adjoint(F, rho, to, gB)
    gFo = gFo.data if sp.issparse(gFo) else np.asarray(gFo)
    for a, b in ((B, Bo), (gE, gEo), (grho, grhoo), (gF, gFo)):
        assert rel_err(a.cpu().numpy(), np.asarray(b).reshape(a.shape)) < TOL
    again = g.transport_backward(ff, tape, dev(rho), dev(gB))
    assert torch.equal(gE, again[0]) and torch.equal(grho, again[1]) and torch.equal(gF, again[2])


def test_idle_lanes_bring_no_infinity_of_another_coefficient(g):
    """Lanes past a chunk read its last coefficient again: what is not finite
    there stays in its own coefficient and colour."""
    n = 300
    rp, col, val = _operator(n, LENGTHS["few"], seed=3)
    E = scenes.seeded_array((n, 17, 1, 3), 2)
    E[40, 8, 0, 1] = np.inf     # the last coefficient of the first of two chunks of nine
    rho = scenes.seeded_array((n, 3), 1, 0.2, 0.9)
    ff = g.ff_from_csr(dev(rp), dev(col), dev(val))
    B, tape = g.transport_solve(ff, dev(rho), dev(E), 1)
    gE, grho, gF = g.transport_backward(ff, tape, dev(rho), dev(scenes.seeded_array((n, 17, 1, 3), 4, 0.1, 1.0)))
    hit = np.array([40 in col[rp[i]:rp[i + 1]] for i in range(n)])
    want = np.zeros((n, 17, 1, 3), bool)
    want[hit, 8, 0, 1] = want[40, 8, 0, 1] = True
    assert np.array_equal(~np.isfinite(B.cpu().numpy()), want)
    assert np.isfinite(gE.cpu().numpy()).all()
    bad = ~np.isfinite(grho.cpu().numpy())
    assert np.array_equal(bad[:, 1], hit) and not bad[:, [0, 2]].any()
    assert np.array_equal(~np.isfinite(gF.cpu().numpy()), col == 40)
