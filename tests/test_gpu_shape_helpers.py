"""Cells whose search for the largest node distance is shared by several
workgroups (cm_shape) on the GPU: spheres, of whose candidates all remain, on
both sides of the counts from which the pairs are shared, with the largest
number of cells and one more, beside cells of few remaining nodes, with an
inverted tetrahedron and non-finite positions, and again and again on one handle
(the arrival counters return to zero).  d_max is a maximum of float64 distances
of float32 positions: 1e-14 relative against numpy's."""
import time

import numpy as np
import pytest
from scipy.spatial import ConvexHull
from scipy.spatial.distance import pdist

from gpu_util import require_gpu
from synth.configs import paper_sphere_case
from synth.mesh import fibonacci_sphere, orient_positive

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _star(surface):
    """A ball of tetrahedra about one interior node: every other node is a
    candidate."""
    p = fibonacci_sphere(surface)
    tri = ConvexHull(p).simplices
    x = np.concatenate([np.zeros((1, 3)), p])
    tets = np.concatenate([np.zeros((len(tri), 1), int), tri + 1], axis=1).astype(np.int32)
    return x, orient_positive(x, tets)


def _d_max(p):
    return pdist(p.astype(np.float64)).max()


def _same(a, b):
    assert abs(a - b) <= 1e-14 * b


@pytest.mark.parametrize("cells", [1, 3, 256, 257])
@pytest.mark.parametrize("surface", [300, 768, 769, 1500])
def test_spheres(surface, cells):
    from paper_2003_03130_amd import CellBatch
    x, tets = _star(surface)
    cb = CellBatch.template(cells, x, tets)
    scale = 1.0 + 0.01 * (np.arange(cells) % 5)
    y = (x[None] * scale[:, None, None]).astype(np.float32)
    out = cb.shape(cb.to_device(y.reshape(-1, 3)), 2.0).cpu().numpy()
    for k in range(min(cells, 5)):
        _same(out[k, 8], _d_max(y[k]))
        assert abs(out[k, 9] - (out[k, 8] - 2.0) / 2.0) <= 1e-15
        assert np.array_equal(out[k::5, 8], np.full(len(out[k::5]), out[k, 8]))
    # rings of a few nodes to most of them remain
    y[:, :, 2] *= np.linspace(0.95, 1.0, cells, dtype=np.float32)[:, None]
    out = cb.shape(cb.to_device(y.reshape(-1, 3)), 2.0).cpu().numpy()
    for k in np.unique(np.linspace(0, cells - 1, 12).astype(int)):
        _same(out[k, 8], _d_max(y[k]))


@pytest.mark.parametrize("cells", [1, 40])
def test_at_the_most_candidates(cells):
    from paper_2003_03130_amd import CellBatch
    x, tets = _star(4096)
    cb = CellBatch.template(cells, x, tets)
    y = np.tile(x, (cells, 1)).astype(np.float32)
    out = cb.shape(cb.to_device(y), 2.0).cpu().numpy()
    d = _d_max(x.astype(np.float32))
    for k in range(cells):
        _same(out[k, 8], d)


def test_uneven_cells_again_and_again():
    """A sphere whose pairs are shared, a small one, an elongated cell, a flat
    one; all fields are the same at every call, also after calls in which
    another cell's pairs are shared."""
    from paper_2003_03130_amd import CellBatch
    stars = [_star(n) for n in (1500, 100, 900, 2000)]
    off = np.concatenate([[0], np.cumsum([len(x) for x, _ in stars])])
    toff = np.concatenate([[0], np.cumsum([len(t) for _, t in stars])])
    x = np.concatenate([s[0] for s in stars])
    cb = CellBatch(off, toff, x, np.concatenate([s[1] for s in stars]))
    forms = np.array([[1, 1, 1], [1, 1, 1], [2, 1, 1], [1, 1, 0.3]])
    outs = []
    for shift in (0, 1, 0, 2, 3, 0):
        f = np.roll(forms, shift, axis=0)
        y = np.concatenate([s[0] * f[k] for k, s in enumerate(stars)]).astype(np.float32)
        out = cb.shape(cb.to_device(y), 2.0).cpu().numpy()
        for k in range(len(stars)):
            _same(out[k, 8], _d_max(y[off[k]:off[k + 1]]))
        if shift == 0:
            outs.append(out)
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


@pytest.mark.parametrize("small", [300, 1000])
def test_large_cells_among_many(small):
    """Two large spheres among many small cells, for which the shared search has a
    launch of its own or goes beside the cells' fields."""
    from paper_2003_03130_amd import CellBatch
    stars = [_star(20)] * (small // 2) + [_star(3700)] + [_star(20)] * (small // 2) + [_star(2500)]
    off = np.concatenate([[0], np.cumsum([len(x) for x, _ in stars])])
    toff = np.concatenate([[0], np.cumsum([len(t) for _, t in stars])])
    x = np.concatenate([s[0] for s in stars])
    cb = CellBatch(off, toff, x, np.concatenate([s[1] for s in stars]))
    for f in ([1, 1, 1], [1.3, 1, 0.9]):
        y = (x * f).astype(np.float32)
        out = cb.shape(cb.to_device(y), 2.0).cpu().numpy()
        for k in (0, small // 2, small // 2 + 1, len(stars) - 1):
            _same(out[k, 8], _d_max(y[off[k]:off[k + 1]]))


def test_inverted_and_non_finite():
    from paper_2003_03130_amd import CellBatch
    x, tets = _star(800)
    cb = CellBatch.template(3, x, tets)
    y = np.tile(x, (3, 1)).reshape(3, -1, 3).astype(np.float32)
    y[0, 0] = [0.0, 0.0, 9.0]   # the hub, no candidate, far outside
    y[1, 0] = np.nan            # its distances are no number
    y[2, 0] = [0.0, np.inf, 0.0]
    out = cb.shape(cb.to_device(y.reshape(-1, 3)), 2.0).cpu().numpy()
    _same(out[0, 8], _d_max(y[0]))
    _same(out[1, 8], _d_max(y[1, 1:]))
    assert out[2, 8] == np.inf
    y[:, 0] = 0.0
    y[1, 5] = np.nan            # a candidate
    y[2, 7] = [-np.inf, 0.0, 0.0]
    out = cb.shape(cb.to_device(y.reshape(-1, 3)), 2.0).cpu().numpy()
    _same(out[0, 8], _d_max(y[0]))
    _same(out[1, 8], _d_max(np.delete(y[1], 5, axis=0)))
    assert out[2, 8] == np.inf


def test_a_sphere_takes_about_the_time_of_an_ellipsoid():
    """One workgroup that compared all pairs of a sphere of 20,000 nodes took ten
    times as long as for an ellipsoid; shared among workgroups they take two to
    three times as long."""
    import torch
    from paper_2003_03130_amd import CellBatch
    c = paper_sphere_case(2003)
    cb = CellBatch.single(c.x, c.tets)
    ys = [cb.to_device((c.x / np.linalg.norm(c.x, axis=1).max() * f).astype(np.float32))
          for f in ([1, 1, 1], [1.2, 1, 0.9])]
    out = cb.shape(ys[0], 2.0)
    us = []
    for y in ys:
        best = np.inf
        for _ in range(10):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(20):
                cb.shape(y, out=out)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        us.append(best / 20 * 1e6)
    assert us[0] < 6.0 * us[1], us
