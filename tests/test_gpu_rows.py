"""The FP32 row products at the edges of their layouts: coefficients that
fill one lane, a quad, a row of 16 lanes or more than one chunk, rows whose
entries end at, before and after a reading of 64, and more bounces than one
launch of the sampled products takes."""
import numpy as np
import pytest
import scipy.sparse as sp

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, rel_err  # noqa: E402

# FP32 sums of up to 200 products of values in [0, 1]: 200 x 2^-24 of the
# largest sum bounds one product's error, nine bounces carry nine of them
TOL = 9 * 200 * 2.0 ** -24

LENGTHS = [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 200]


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


@pytest.fixture(scope="module")
def orc():
    import oracle as o
    return o


def _operator(n, seed):
    rng = np.random.default_rng(seed)
    lens = np.resize(LENGTHS, n)
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(lens)
    col = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lens]).astype(np.int32)
    val = (rng.uniform(0.1, 1.0, col.size) * np.repeat(0.6 / np.maximum(lens, 1), lens)).astype(np.float32)
    return rp, col, val


@pytest.mark.parametrize("lights,K", [(1, 1), (1, 4), (5, 1), (1, 16), (17, 1), (33, 1)])
@pytest.mark.parametrize("n,nb", [(203, 1), (230, 9)])
def test_row_products_at_layout_edges(g, orc, lights, K, n, nb):
    rp, col, val = _operator(n, seed=lights + K)
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


def test_a_value_that_is_not_finite_stays_in_its_colour(g):
    """Lanes past a row's columns and entries past a row's end do not bring
    another row's infinity into a sum, and no colour another's."""
    n = 210
    rp, col, val = _operator(n, seed=3)
    E = scenes.seeded_array((n, 1, 9, 3), 2)
    E[40, 0, 0, 0] = np.inf          # red, the coefficient that idle lanes read
    rho = scenes.seeded_array((n, 3), 1, 0.2, 0.9)
    ff = g.ff_from_csr(dev(rp), dev(col), dev(val))
    B, tape = g.transport_solve(ff, dev(rho), dev(E), 1)
    gE, grho, gF = g.transport_backward(ff, tape, dev(rho), dev(scenes.seeded_array((n, 1, 9, 3), 4, 0.1, 1.0)))
    hit = np.array([40 in col[rp[i]:rp[i + 1]] for i in range(n)])
    bad = ~np.isfinite(B.cpu().numpy())
    want = np.zeros_like(bad)
    want[hit, 0, 0, 0] = True
    want[40, 0, 0, 0] = True
    assert np.array_equal(bad, want)
    assert np.isfinite(gE.cpu().numpy()).all()
    bad = ~np.isfinite(grho.cpu().numpy())
    assert np.array_equal(bad[:, 0], hit) and not bad[:, 1:].any()
    assert np.array_equal(~np.isfinite(gF.cpu().numpy()), col == 40)
