"""The search for a cell's largest node distance by one workgroup (cm_shape) on
the GPU: spheres (every candidate remains), flat, elongated and sheared cells,
few nodes, cells with an inverted tetrahedron, non-finite positions, and cells
on both sides of the candidate count at which the search goes over blocks
instead.  d_max is a maximum of float64 distances of float32 positions: 1e-14
relative against numpy's."""
import numpy as np
import pytest
from scipy.spatial import ConvexHull
from scipy.spatial.distance import pdist

from gpu_util import require_gpu
from synth.configs import paper_sphere_case, small_sphere_case
from synth.mesh import fibonacci_sphere, orient_positive

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _d_max(p):
    # the farthest pair are hull vertices
    p = p.astype(np.float64)
    if len(p) > 64:
        p = p[ConvexHull(p).vertices]
    return pdist(p).max()


def _shape(cb, y):
    return cb.shape(cb.to_device(y), 2.0).cpu().numpy()


def _same(a, b):
    assert abs(a - b) <= 1e-14 * b


@pytest.mark.parametrize("form", [(1, 1, 1), (1, 1, 0.2), (2, 1, 0.7), (3, 0.3, 0.3),
                                  (1, 1, 1.0001)])
@pytest.mark.parametrize("seed", [1000, 1006])
def test_forms(form, seed):
    from paper_2003_03130_amd import CellBatch
    c = small_sphere_case(seed)
    rng = np.random.default_rng(seed)
    Q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    copies = 5
    cb = CellBatch.template(copies, c.x, c.tets)
    y = np.concatenate([(c.x * np.array(form) * (1 + 0.1 * k)) @ Q + [3.0, -1.0, 0.5 * k]
                        for k in range(copies)]).astype(np.float32)
    out = _shape(cb, y)
    n = len(c.x)
    for k in range(copies):
        _same(out[k, 8], _d_max(y[k * n:(k + 1) * n]))
        assert abs(out[k, 9] - (out[k, 8] - 2.0) / 2.0) <= 1e-15


def test_a_single_tetrahedron_and_one_point():
    from paper_2003_03130_amd import CellBatch
    x = np.array([[0.0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]])
    cb = CellBatch.single(x, np.array([[0, 1, 2, 3]]))
    _same(_shape(cb, x.astype(np.float32))[0, 8], np.sqrt(2.0))
    # all nodes at one point: distance 0 (and no volume)
    assert _shape(cb, np.full((4, 3), 0.25, np.float32))[0, 8] == 0.0


def test_inverted_cells():
    """All nodes are searched: an interior node moved out through the surface
    (and its tetrahedra inside out) is found."""
    from paper_2003_03130_amd import CellBatch
    for c in (small_sphere_case(1002), paper_sphere_case(2004)):
        cb = CellBatch.single(c.x, c.tets)
        y = c.x.astype(np.float32)
        inner = int(np.argmin(np.linalg.norm(c.x, axis=1)))
        y[inner] = [0.0, 0.0, 9.0]
        out = _shape(cb, y)[0]
        _same(out[8], _d_max(y))


def test_non_finite_positions():
    from paper_2003_03130_amd import CellBatch
    c = small_sphere_case(1004)
    cb = CellBatch.single(c.x, c.tets)
    y = c.x.astype(np.float32)
    inner = int(np.argmin(np.linalg.norm(c.x, axis=1)))
    y[inner] = np.nan  # its distances are no number; the others' maximum remains
    _same(_shape(cb, y)[0, 8], _d_max(np.delete(y, inner, axis=0)))
    y[inner] = [np.inf, 0.0, 0.0]
    assert _shape(cb, y)[0, 8] == np.inf


@pytest.mark.parametrize("surface", [4096, 4098, 8194])
def test_candidates_at_the_limit(surface):
    """A star of tetrahedra about one interior node: every surface node is a
    candidate; 4,096 are the most that one workgroup searches."""
    from paper_2003_03130_amd import CellBatch
    p = fibonacci_sphere(surface) * [1.0, 1.05, 0.9]
    tri = ConvexHull(p).simplices
    x = np.concatenate([np.zeros((1, 3)), p])
    tets = np.concatenate([np.zeros((len(tri), 1), int), tri + 1], axis=1).astype(np.int32)
    cb = CellBatch.single(x, orient_positive(x, tets))
    y = (x @ np.array([[1.0, 0.2, 0], [0, 1.1, 0.1], [0, 0, 0.8]])).astype(np.float32)
    _same(_shape(cb, y)[0, 8], _d_max(y))
