"""Form factors over trees whose walks need more stack than lies in LDS."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev_surfels, gpu_csr, rel_err  # noqa: E402

TOL = 1e-4   # of the largest value, as the other form factor tests


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


@pytest.mark.parametrize("copies", [4, 7])
def test_deep_trees_are_traced_once(g, orc, copies):
    """Every box of a chain of 31 nodes is open at once; the rays cross fewer
    surfels than they have record slots, so one trace is enough."""
    sur = scenes.deep_chain(copies=copies)
    bvh = g.build_bvh(dev_surfels(sur))
    assert bvh.height() >= 32 and sur["px"].shape[0] < 256
    g.profile_enable(True)
    try:
        ff = g.form_factors(bvh, 32, 3, t_min=1e-4)
        torch.cuda.synchronize()
        rep = g.profile_report()
    finally:
        g.profile_enable(False)
    assert rep["ff_trace"]["count"] == 1
    F = gpu_csr(ff)
    Fo, _ = orc.ff_matrix(sur, 32, 3, orc.default_t_eps(sur), 1e-4, 0)
    assert np.array_equal(F.indptr, Fo.indptr) and np.array_equal(F.indices, Fo.indices)
    assert rel_err(F.data, Fo.data) < TOL


def test_deep_subtrees(g, orc):
    """64 surfels at every centre: entries are set aside more than once."""
    sur = scenes.deep_chain(copies=64, opacity=0.5)
    F = gpu_csr(g.form_factors(g.build_bvh(dev_surfels(sur)), 4, 3, t_min=1e-4))
    Fo, _ = orc.ff_matrix(sur, 4, 3, orc.default_t_eps(sur), 1e-4, 0)
    assert np.array_equal(F.indptr, Fo.indptr) and np.array_equal(F.indices, Fo.indices)
    assert rel_err(F.data, Fo.data) < TOL
