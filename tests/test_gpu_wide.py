"""Tile passes with several wavefronts per tile (the default launch: node
lists up to 256 tiles, turns beyond) against the one-wavefront passes
(cm_set_launch with a persistent grid) on the GPU: forces, energies, counts,
ybar, parameter gradients, Hessian-vector products and plate steps must be
equal bit for bit -- every addition keeps its place -- for tiles of one chunk
(fewer than wavefronts), of 2 to 17 chunks and more, and on both sides of the
tile counts at which the pass or its number of wavefronts changes.  The
one-wavefront passes are held to the FP64 oracle by the forward, backward and
fused tests."""
import numpy as np
import pytest

from gpu_util import require_gpu
from synth.configs import cotangent, radial_regions, random_theta, small_sphere_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _all_passes(cb, y, fb, eb, plate):
    import torch
    from paper_2003_03130_amd import _native as nat
    from paper_2003_03130_amd.cells import _ptr, _stream
    nan = float("nan")
    out = {}
    ninv = torch.full((cb.n_cells,), -1, dtype=torch.int32, device=cb.device)
    f, E, nonfin = cb.forces_checked(y, n_inverted=ninv)
    out.update(f=f, E=E, ninv=ninv, nonfin=nonfin)
    out["ybar"], out["thetabar"] = cb.backward(y, fb, eb)
    hvp = cb.empty_nodes().fill_(nan)
    nat.check(nat.lib().cm_forces_backward(cb._h, _ptr(y), _ptr(fb), None, _ptr(hvp),
                                           None, _stream(None)))
    out["hvp"] = hvp
    out["f2"], out["E2"], out["ybar2"], out["thetabar2"] = cb.forces_and_backward(y, fb, eb)
    y1, lam = cb.empty_nodes().fill_(nan), cb.empty_nodes().fill_(nan)
    force = torch.full((cb.n_cells,), nan, dtype=torch.float64, device=cb.device)
    cb.plate_forces_step(y, plate, 100.0, 4e-3, y1, force)
    tacc = torch.zeros(3 * cb.n_mat, dtype=torch.float64, device=cb.device)
    cb.plate_backward_step(y, fb, plate, 100.0, 4e-3, lam, force, 0.5 * force, 1e-2, tacc)
    out.update(y1=y1, force=force, lam=lam, tacc=tacc)
    torch.cuda.synchronize()
    return out


def _compare(cb, y_host, seed):
    import torch
    y, fb = cb.to_device(y_host), cb.to_device(cotangent(len(y_host), seed))
    eb = torch.linspace(-0.5, 1.5, cb.n_cells, dtype=torch.float64, device=cb.device)
    # plates inside the cells, so that some nodes touch each of them
    z = np.asarray(y_host)[:, 2]
    plate = torch.tensor([0.8 * z.max(), 0.8 * z.min()], dtype=torch.float64,
                         device=cb.device).repeat(cb.n_cells)
    got = _all_passes(cb, y, fb, eb, plate)
    cb.set_launch(1, 1)
    want = _all_passes(cb, y, fb, eb, plate)
    for k, w in want.items():
        assert torch.equal(got[k], w), f"{k} differs"
    assert torch.equal(got["f2"], got["f"]) and torch.equal(got["ybar2"], got["ybar"])


@pytest.mark.parametrize("tile", [64, 128, 192, 320, 768, 1024, 2048])
def test_one_cell(tile):
    from paper_2003_03130_amd import CellBatch
    c = small_sphere_case(1003)
    cb = CellBatch.single(c.x, c.tets, tile_tets=tile)
    cb.set_params(*c.theta)
    _compare(cb, c.y, 1004)


def test_a_single_tetrahedron():
    from paper_2003_03130_amd import CellBatch
    x = np.array([[0.0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]])
    cb = CellBatch.single(x, np.array([[0, 1, 2, 3]]))
    cb.set_params(1.0, 10.0, 0.5)
    y = (x * [0.9, 1.1, 0.8] + 0.01 * np.arange(12).reshape(4, 3)).astype(np.float32)
    _compare(cb, y, 5)


def test_regions():
    from paper_2003_03130_amd import CellBatch
    c = small_sphere_case(1005)
    cb = CellBatch.single(c.x, c.tets, regions=radial_regions(c.x, c.tets), n_regions=3)
    th = np.array([random_theta(np.random.default_rng(k)) for k in range(3)])
    cb.set_params(*th.T)
    _compare(cb, c.y, 1006)


@pytest.mark.parametrize("tile", [64, 128, 192, 320, 768, 1024])
def test_few_chunks_a_tile_in_turns(tile):
    """As test_one_cell with more than 256 tiles: the turns' tiles of one
    chunk and more."""
    from paper_2003_03130_amd import CellBatch
    c = small_sphere_case(1003)
    n = CellBatch.single(c.x, c.tets, tile_tets=tile).info["n_tiles"]
    copies = 256 // n + 1
    cb = CellBatch.template(copies, c.x, c.tets, tile_tets=tile)
    assert 256 < cb.info["n_tiles"] <= 1536
    cb.set_params(*c.theta)
    _compare(cb, np.tile(c.y, (copies, 1)), 1004)


# 12 tiles a copy: 252 and 264 tiles (lists up to 256), 1,536 and 1,548 (four
# wavefronts up to 1,536), 6,492 and 6,504 (four up to 6,500 for the
# Hessian-vector product)
@pytest.mark.parametrize("copies", [21, 22, 128, 129, 541, 542])
def test_tile_counts_where_the_wavefronts_change(copies):
    from paper_2003_03130_amd import CellBatch
    c = small_sphere_case(1000)
    cb = CellBatch.template(copies, c.x, c.tets, tile_tets=448)
    assert cb.info["n_tiles"] == 12 * copies
    rng = np.random.default_rng(copies)
    cb.set_params(*np.array([random_theta(rng) for _ in range(copies)]).T)
    y = np.tile(c.y, (copies, 1)) * rng.uniform(0.95, 1.05, (copies * len(c.y), 1))
    _compare(cb, y.astype(np.float32), copies)
