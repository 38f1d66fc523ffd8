"""cm_profile_kernels on the GPU times the launches that an evaluation makes: no
finalize where the tile pass forms the cells' sums itself, which depends on the
tiles, the cells' shared nodes and the launch shape; the timed launches leave the
outputs of an evaluation."""
import numpy as np
import pytest

from gpu_util import require_gpu
from synth.configs import cotangent
from synth.mesh import sphere_mesh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# nodes of the cell, cells, launch -> whether forward, backward and both passes
# at once have a finalize launch (135 and 1,171 shared nodes a cell; more than 256
# tiles; a launch shape of the one-wavefront passes)
@pytest.mark.parametrize("n,cells,launch,finalize", [
    (400, 2, (1, 0), (False, False, False)),
    (2200, 3, (1, 0), (False, False, True)),
    (400, 200, (1, 0), (True, True, True)),
    (400, 2, (1, 1), (True, True, True))])
def test_launches_of_an_evaluation(n, cells, launch, finalize):
    import torch
    from paper_2003_03130_amd import CellBatch
    x, tets = sphere_mesh(n, n)
    cb = CellBatch.template(cells, x, tets)
    cb.set_params(np.full(cells, 1.2), np.full(cells, 15.0), np.full(cells, 0.4))
    cb.set_launch(*launch)
    y = cb.to_device(np.tile(x * 0.95, (cells, 1)).astype(np.float32))
    fb = cb.to_device(cotangent(cb.n_nodes, 3))
    eb = torch.linspace(-1.0, 1.0, cells, dtype=torch.float64, device=cb.device)
    want = cb.forces_and_backward(y, fb, eb)
    got = [torch.full_like(w, -7.0) for w in want]
    f, E, yb, tb = got
    ms = cb.profile_kernels(y, f, E, fb, eb, yb, tb, reps=3)
    assert np.isfinite(ms).all() and (ms[::2] > 0).all()
    assert tuple(ms[1::2] > 0) == finalize, ms
    assert (ms[1::2] >= 0).all()
    for g, w in zip(got, want):
        assert torch.equal(g, w)
