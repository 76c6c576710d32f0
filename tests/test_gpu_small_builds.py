"""Trees built by one workgroup and by many: F against the oracle for surfel
counts at and past the sizes where the sort and the refit change, among them
surfels with equal Morton codes (a stable order)."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, dev_surfels, gpu_csr, rel_err  # noqa: E402

TOL = 1e-4   # of the largest value, as the other form factor tests


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


@pytest.mark.parametrize("n", [2, 63, 65, 1024, 1025, 2047, 2048, 2049, 4096, 4097])
def test_form_factors_at_build_sizes(g, orc, n):
    sur = dict(scenes.random_frame_surfels(n, seed=n, scale=(0.02, 0.08)))
    for a in "xyz":   # every fourth surfel on its neighbour's centre
        sur["p" + a] = sur["p" + a].copy()
        sur["p" + a][3::4] = sur["p" + a][2::4][:sur["p" + a][3::4].size]
    bvh = g.build_bvh(dev_surfels(sur))
    F = gpu_csr(g.form_factors(bvh, 8, 3, t_min=1e-4))
    Fo, _ = orc.ff_matrix(sur, 8, 3, orc.default_t_eps(sur), 1e-4, 0)
    assert np.array_equal(F.indptr, Fo.indptr) and np.array_equal(F.indices, Fo.indices)
    if Fo.nnz:
        assert rel_err(F.data, Fo.data) < TOL
    assert 0 < bvh.height() < 62


@pytest.mark.parametrize("nnz", [1, 300, 4096, 4097])
def test_transpose_at_sort_sizes(g, nnz):
    """dL/dE through F^T against FP64: the transpose sorts nnz columns."""
    import scipy.sparse as sp
    n = 70
    rng = np.random.default_rng(nnz)
    at = np.sort(rng.choice(n * n, nnz, replace=False))
    ptr = np.searchsorted(at, np.arange(n + 1) * n).astype(np.int64)
    col, val = (at % n).astype(np.int32), rng.uniform(0.0, 1.0 / n, nnz).astype(np.float32)
    F = sp.csr_matrix((val.astype(np.float64), col, ptr), shape=(n, n))
    ff = g.ff_from_csr(dev(ptr), dev(col), dev(val))
    rho = scenes.seeded_array((n, 3), 1, 0.2, 0.9)
    E, gB = scenes.seeded_array((n, 1, 4, 3), 2), scenes.seeded_array((n, 1, 4, 3), 3, -1, 1)
    _, tape = g.transport_solve(ff, dev(rho), dev(E), 2)
    gE = g.transport_backward(ff, tape, dev(rho), dev(gB))[0].cpu().numpy()
    want = lam = gB.astype(np.float64)
    for _ in range(2):
        lam = (F.T @ (rho[:, None, None, :] * lam).reshape(n, -1)).reshape(gB.shape)
        want = want + lam
    assert rel_err(gE, want) < 1e-5   # two FP32 sums of at most 70 products
