"""Opacity and geometry gradients whose contributions are listed by block of
surfels, at the edges of the lists: one block and one surfel more, batches of
rays that do not fill a workgroup, rays beyond one batch, and more hits than
the lists hold."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_common import dev, dev_surfels, gpu_csr, rel_err  # noqa: E402
from tests.test_gpu_walks import _sheets  # noqa: E402

TOL = 1e-4   # of the largest value: FP32 terms, 64-bit fixed-point sums


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


def _faced_sheets():
    """Wide sheets of either face: a ray crosses more than 64 of them."""
    sur = _sheets(0, 0, 449)
    for a in "xyz":
        sur["n" + a][::2] *= -1
    return sur


@pytest.mark.parametrize("scene,n,R", [("fruit_bowl", 512, 128), ("fruit_bowl", 513, 128), ("fruit_bowl", 700, 100),
                                       ("box_room", 300, 320), ("fruit_bowl", 4097, 17), ("sheets", 450, 192)])
def test_listed_gradients_match_oracle(g, orc, scene, n, R):
    sur = _faced_sheets() if scene == "sheets" else scenes.make_config(scene, n=n).surfels
    n = sur["px"].shape[0]
    assert n * R >= 1 << 16   # listed
    bvh = g.build_bvh(dev_surfels(sur))
    ff = g.form_factors(bvh, R, 5, t_min=1e-4)
    F = gpu_csr(ff)
    gF = np.random.default_rng(2).standard_normal(F.nnz).astype(np.float32)
    rows, te = (F.indptr, F.indices, gF.astype(np.float64)), orc.default_t_eps(sur)
    alb = np.full((n, 3), 0.5, np.float32)
    got = g.geometry_backward(bvh, ff, dev(gF))
    go, _ = g.opacity_backward(bvh, ff, dev(gF), None, None)
    ref = orc.geometry_backward(sur, R, 5, te, 1e-4, rows)
    rgo = orc.opacity_backward(sur, alb, R, 5, te, 1e-4, rows)[0]
    assert rel_err(go.cpu().numpy(), rgo) < TOL
    for f in orc.GEOMETRY_FIELDS:
        assert rel_err(got[f].cpu().numpy(), ref[f]) < TOL, f
    again = g.geometry_backward(bvh, ff, dev(gF))
    assert torch.equal(g.opacity_backward(bvh, ff, dev(gF), None, None)[0], go)
    for f in orc.GEOMETRY_FIELDS:
        assert torch.equal(got[f], again[f]), f
