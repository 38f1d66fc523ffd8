"""The block search for the largest node distance (cm_shape with a cell of more
than 4,096 candidates) on the GPU over batches: cells on both sides of that count
together, each inverted in turn so that its farthest pair is found among all its
nodes only, and copies of one shared mesh.  (test_gpu_shape.py has the search by
one workgroup per cell: its largest mesh has 2,477 candidates.)  Against the
float64 oracle, with the tolerances of float64 rounding given there."""
import numpy as np
import pytest

from gpu_util import require_gpu
from oracle import shape as oshape
from scipy.spatial import ConvexHull
from synth.configs import small_sphere_case
from synth.mesh import fibonacci_sphere, orient_positive

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _star(surface):
    """A ball of tetrahedra about one interior node (the first): every other
    node is a candidate."""
    p = fibonacci_sphere(surface) * [1.0, 1.05, 0.9]
    tri = ConvexHull(p).simplices
    x = np.concatenate([np.zeros((1, 3)), p])
    tets = np.concatenate([np.zeros((len(tri), 1), int), tri + 1], axis=1).astype(np.int32)
    return x, orient_positive(x, tets)


def _check(r, x, y, tets, d_ref, inverted=False):
    ref = oshape.cell_shape(x, y.astype(np.float64), tets, d_ref)
    assert abs(r[8] - ref["d_max"]) <= 1e-12 * ref["d_max"]
    assert abs(r[9] - ref["strain"]) <= 1e-12 * max(1.0, abs(ref["strain"]))
    if inverted:  # (volumes of both signs: no rounding bar from their sum)
        return
    assert abs(r[0] - ref["volume"]) <= 1e-12 * abs(ref["volume"])
    assert np.abs(r[1:4] - ref["com"]).max() <= 1e-12 * np.abs(y).max()
    assert np.abs(r[4:7] - ref["axes"]).max() <= 1e-10 * ref["axes"].max()
    assert abs(r[7] - ref["D"]) <= 1e-10


def test_batch_of_cells_about_the_limit():
    from paper_2003_03130_amd import CellBatch
    small = [small_sphere_case(s) for s in (1001, 1003)]
    cells = [(small[0].x, small[0].tets), _star(4098), (small[1].x, small[1].tets),
             _star(4500), _star(300)]
    off = np.concatenate([[0], np.cumsum([len(x) for x, _ in cells])])
    toff = np.concatenate([[0], np.cumsum([len(t) for _, t in cells])])
    x = np.concatenate([c[0] for c in cells])
    tets = np.concatenate([c[1] for c in cells])
    cb = CellBatch(off, toff, x, tets)
    d_ref = np.linspace(1.8, 2.2, len(cells))
    A = np.array([[1.0, 0.2, 0.0], [0.0, 1.1, 0.1], [0.0, 0.0, 0.8]])
    base = (x @ A + [3.0, -2.0, 1.0]).astype(np.float32)
    # upright, then each cell with the node nearest to its centre (no candidate)
    # far outside: one end of its farthest pair
    for turned in [None, *range(len(cells))]:
        y = base.copy()
        if turned is not None:
            s = slice(off[turned], off[turned + 1])
            inner = off[turned] + int(np.argmin(np.linalg.norm(x[s], axis=1)))
            y[inner] = [3.0, -2.0 + 0.5 * turned, 8.0]
        out = cb.shape(cb.to_device(y), d_ref).cpu().numpy()
        for c in range(len(cells)):
            s, t = slice(off[c], off[c + 1]), slice(toff[c], toff[c + 1])
            _check(out[c], x[s], y[s], tets[t], d_ref[c], inverted=c == turned)
        if turned is not None:
            assert out[turned, 8] > 5.0  # (the cells' own extent is below 3)


def test_copies_of_a_shared_mesh():
    from paper_2003_03130_amd import CellBatch
    x, tets = _star(4200)
    cb = CellBatch.template(2, x, tets)
    y = np.concatenate([x * [1.0, 1.0, 0.7], x * [0.6, 1.3, 1.0] + 2.0]).astype(np.float32)
    n = len(x)
    for turned in (None, 1, 0):
        yt = y.copy()
        if turned is not None:
            yt[turned * n] = [0.0, 7.0, 0.0]
        out = cb.shape(cb.to_device(yt), 2.0).cpu().numpy()
        for c in range(2):
            _check(out[c], x, yt[c * n:(c + 1) * n], tets, 2.0, inverted=c == turned)
