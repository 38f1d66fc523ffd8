"""Sums of a cell by the workgroup that finishes its last tile (tile passes of
up to 256 tiles whose cells have up to 2,048 shared nodes, both passes at once
up to 512) on the GPU: every output bit for bit that of the one-wavefront
passes with their finalize launch (cm_set_launch), for cells on both sides of
those limits, uneven cells in one batch, nodes of no tetrahedron, material
regions, inactive cells, per-cell launches, and over repeated calls with a
forward and a backward, or a forward and one without the handle's scratch, side
by side on two streams."""
import numpy as np
import pytest

from gpu_util import require_gpu
from synth.configs import cotangent, radial_regions, random_theta, small_sphere_case
from synth.mesh import sphere_mesh
from test_gpu_wide import _compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _ball(n):
    x, tets = sphere_mesh(n, n)
    rng = np.random.default_rng(n)
    y = x * rng.uniform(0.9, 1.1, 3) + rng.normal(0, 2e-3, x.shape)
    return x, tets, y.astype(np.float32)


def _batch(parts, **kw):
    from paper_2003_03130_amd import CellBatch
    off = [np.concatenate([[0], np.cumsum([len(p[k]) for p in parts])]) for k in (0, 1)]
    return CellBatch(*off, np.concatenate([p[0] for p in parts]),
                     np.concatenate([p[1] for p in parts]), **kw)


@pytest.mark.parametrize("n", [400, 1000, 1500, 2200, 3600, 4600])
def test_shared_nodes_about_the_limits(n):
    p = _ball(n)
    cb = _batch([p])
    cb.set_params(1.2, 15.0, 0.4)
    _compare(cb, p[2], n)


def test_uneven_cells_and_loose_nodes():
    parts = [_ball(n) for n in (300, 1800, 60, 900)]
    loose = np.array([[5.0, 0.0, 0.9], [5.0, 1.0, -0.9]])
    parts[1] = (np.concatenate([parts[1][0], loose]), parts[1][1],
                np.concatenate([parts[1][2], loose.astype(np.float32)]))
    reg = np.concatenate([radial_regions(p[0], p[1]) for p in parts])
    cb = _batch(parts, regions=reg, n_regions=3)
    rng = np.random.default_rng(3)
    cb.set_params(*np.array([random_theta(rng) for _ in range(cb.n_mat)]).T)
    _compare(cb, np.concatenate([p[2] for p in parts]), 7)


def test_inactive_cells_and_percell_launches():
    import torch
    parts = [_ball(n) for n in (500, 1200, 700, 900)]
    cb = _batch(parts)
    cb.set_params(1.0, 20.0, 0.3)
    y = cb.to_device(np.concatenate([p[2] for p in parts]))
    fb = cb.to_device(cotangent(cb.n_nodes, 5))
    f, E = cb.forces(y)
    yb, tb = cb.backward(y, fb)
    for _ in range(2):
        f1, E1 = cb.forces(y, percell=True)
        yb1, tb1 = cb.backward(y, fb, percell=True)
        for a, b in ((f1, f), (E1, E), (yb1, yb), (tb1, tb)):
            assert torch.equal(a, b)
        on = torch.tensor([0.0, 1.0, 0.0, 2.0], dtype=torch.float64, device=cb.device)
        yb2 = torch.full_like(yb, -7.0)
        tb2 = torch.full_like(tb, -7.0)
        cb.backward(y, fb, ybar=yb2, thetabar=tb2, cells=on)
        off = np.asarray(cb.node_off)
        for c in range(4):
            for d in range(3):
                s = slice(d * cb.n_nodes + off[c], d * cb.n_nodes + off[c + 1])
                want = yb[s] if on[c] != 0 else torch.full_like(yb[s], -7.0)
                assert torch.equal(yb2[s], want)
            want = tb[3 * c:3 * c + 3] if on[c] != 0 else torch.full_like(tb[:3], -7.0)
            assert torch.equal(tb2[3 * c:3 * c + 3], want)


def test_repeated_calls_beside_each_other():
    import torch
    from paper_2003_03130_amd import CellBatch
    from paper_2003_03130_amd import _native as nat
    from paper_2003_03130_amd.cells import _ptr, _stream
    c = small_sphere_case(1002)
    cb = CellBatch.template(6, c.x, c.tets, tile_tets=256)
    assert cb.info["n_tiles"] <= 256
    cb.set_params(*c.theta)
    y = cb.to_device(np.tile(c.y, (6, 1)))
    fb = cb.to_device(cotangent(cb.n_nodes, 9))
    cb.set_launch(1, 1)
    f, E = cb.forces(y)
    yb, tb = cb.backward(y, fb)
    cb.set_launch(1, 0)
    torch.cuda.synchronize()
    sides = [torch.cuda.Stream() for _ in range(2)]

    def noalloc():
        g, e = torch.empty_like(f), torch.empty_like(E)
        nat.check(nat.lib().cm_forces_noalloc(cb._h, _ptr(y), _ptr(g), _ptr(e), None,
                                              _stream(None)))
        return g, e

    for beside, want in ((lambda: cb.backward(y, fb), (yb, tb)), (noalloc, (f, E))):
        outs = []
        for _ in range(100):
            with torch.cuda.stream(sides[0]):
                a = cb.forces(y)
            with torch.cuda.stream(sides[1]):
                b = beside()
            outs.append((*a, *b))
        torch.cuda.synchronize()
        for o in outs:
            for got, w in zip(o, (f, E, *want)):
                assert torch.equal(got, w)
