"""The form-factor trace's grid boxes where the grid is coarse or degenerate:
trees of a few nodes, a scene without thickness, far from the origin, with one
surfel a million times further away than the rest is wide, and rays that start
on the scene's box.  Boxes only decide which surfels are tested, so the rows
are the oracle's."""
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


def _scene(kind, n):
    sur = dict(scenes.random_frame_surfels(n, seed=n, scale=(0.1, 0.4)))
    if kind == "flat":
        sur["pz"] = np.zeros_like(sur["pz"])
    elif kind == "far":
        sur["px"] = (sur["px"] + np.float32(3000.0)).astype(np.float32)
        sur["pz"] = (sur["pz"] - np.float32(500.0)).astype(np.float32)
    elif kind == "outlier":
        sur["py"] = sur["py"].copy()
        sur["py"][n // 2] = 1e6
    return sur


@pytest.mark.parametrize("kind,n", [("plain", 2), ("plain", 3), ("plain", 4), ("plain", 5), ("plain", 300),
                                    ("flat", 300), ("far", 300), ("outlier", 300)])
def test_form_factors_on_grid_boxes(g, orc, kind, n):
    sur = _scene(kind, n)
    ff = g.form_factors(g.build_bvh(dev_surfels(sur)), 64, 7, t_min=1e-4)
    F = gpu_csr(ff)
    Fo, _ = orc.ff_matrix(sur, 64, 7, orc.default_t_eps(sur), 1e-4, 0)
    assert np.array_equal(F.indptr, Fo.indptr) and np.array_equal(F.indices, Fo.indices)
    if Fo.nnz:
        assert rel_err(F.data, Fo.data) < TOL
