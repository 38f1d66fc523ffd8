"""Parameters from strided device tensors (cm_set_params_strided) on the GPU:
columns of a (slots, 3) theta, every second entry, one value for all
(stride 0), (cells, regions) tables and other types must give bit for bit the
forces of the same values from the host."""
import ctypes

import numpy as np
import pytest

from gpu_util import require_gpu
from synth.configs import radial_regions, random_theta, small_sphere_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [1, 3, 300])
@pytest.mark.parametrize("form", ["columns", "rows", "spread", "one", "table", "float32"])
def test_strided_parameters(form, copies):
    require_gpu()
    import torch
    from paper_2003_03130_amd import CellBatch
    c = small_sphere_case(1001)
    cb = CellBatch.template(copies, c.x, c.tets, regions=radial_regions(c.x, c.tets),
                            n_regions=3)
    rng = np.random.default_rng(copies)
    th = np.array([random_theta(rng) for _ in range(cb.n_mat)])
    if form == "one":
        th[:] = th[0]
    if form == "float32":
        th = th.astype(np.float32).astype(np.float64)
    y = cb.to_device(np.tile(c.y, (copies, 1)))
    cb.set_params(th[:, 0], th[:, 1], th[:, 2])
    want = [t.clone() for t in cb.forces(y)]
    cb.set_params(1.0, 10.0, 0.5)
    d = torch.from_numpy(th).to(cb.device)
    if form == "columns":
        args = d[:, 0], d[:, 1], d[:, 2]
    elif form == "rows":
        t = d.t().contiguous()
        args = t[0], t[1], t[2]
    elif form == "spread":
        t = torch.full((2 * cb.n_mat, 3), float("nan"), dtype=torch.float64, device=cb.device)
        t[::2] = d
        args = t[::2, 0], t[::2, 1], t[::2, 2]
    elif form == "one":
        args = [d[0, k].expand(cb.n_mat) for k in range(3)]
    elif form == "table":
        args = [d[:, k].reshape(copies, 3) for k in range(3)]
    else:
        args = [d[:, k].float() for k in range(3)]
    cb.set_params(*args)
    for g, w in zip(cb.forces(y), want):
        assert torch.equal(g, w)


def test_refused():
    require_gpu()
    import torch
    from paper_2003_03130_amd import CellBatch, _native as nat
    c = small_sphere_case(1001)
    cb = CellBatch.single(c.x, c.tets)
    t = torch.ones(2, dtype=torch.float64, device=cb.device)
    with pytest.raises(ValueError):
        cb.set_params(t, t, t)
    p = ctypes.c_void_p(t.data_ptr())
    fn = nat.lib().cm_set_params_strided
    assert fn(None, p, 1, p, 1, p, 1, None) == nat.CM_EINVAL
    assert fn(cb._h, None, 1, p, 1, p, 1, None) == nat.CM_EINVAL
    assert fn(cb._h, p, -1, p, 1, p, 1, None) == nat.CM_EINVAL
