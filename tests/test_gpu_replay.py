"""Replays of a captured evaluation (cm_graph_launch) on the GPU: every replay
must give bit for bit what the calls give eagerly, with the parameters and the
buffer contents of its moment, whatever the handle's launch shape has become
since the capture, on the capture's stream or another, and inside an outer
graph capture."""
import pytest

from gpu_util import require_gpu
from synth.configs import cotangent, small_sphere_case

pytestmark = pytest.mark.gpu


def _setup(mode):
    import torch
    from paper_2003_03130_amd import CellBatch
    c = small_sphere_case(1002)
    cb = CellBatch.single(c.x, c.tets)
    cb.set_params(*c.theta)
    y, fb = cb.to_device(c.y), cb.to_device(cotangent(c.n_nodes, 7))
    eb = torch.tensor([0.6], dtype=torch.float64, device=cb.device)
    out = {"f": cb.empty_nodes(), "E": torch.empty(1, dtype=torch.float64, device=cb.device),
           "yb": cb.empty_nodes(), "tb": torch.empty(3, dtype=torch.float64, device=cb.device)}
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    cb.graph_capture(mode, y, out["f"], out["E"], None, fb, eb, out["yb"], out["tb"], stream=st)
    return cb, y, fb, eb, out, st


def _eager(cb, y, fb, eb, mode):
    f, E = cb.forces(y)
    want = {"f": f, "E": E}
    if mode:
        want["yb"], want["tb"] = cb.backward(y, fb, eb)
    return want


@pytest.mark.parametrize("mode", [0, 1, 4, 6])
def test_replays(mode):
    require_gpu()
    import torch
    cb, y, fb, eb, out, st = _setup(mode)
    steps = [None, lambda: cb.set_params(1.7, 21.0, 0.2), lambda: y.mul_(1.01),
             lambda: cb.set_launch(1, 1), lambda: fb.mul_(-2.0), lambda: cb.set_launch(1, 0)]
    for k, change in enumerate(steps):
        if change:
            change()
        want = _eager(cb, y, fb, eb, mode)
        for t in out.values():
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        stream = st if k % 2 else torch.cuda.current_stream()
        cb.graph_launch(stream=stream)
        torch.cuda.synchronize()
        for n, w in want.items():
            assert torch.equal(out[n], w), f"step {k}: {n} differs"


def test_launch_inside_a_capture():
    require_gpu()
    import torch
    cb, y, fb, eb, out, st = _setup(6)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cb.graph_launch()
    for k in range(4):
        y.mul_(1.0 + 0.01 * k)
        want = _eager(cb, y, fb, eb, 6)
        for t in out.values():
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for n, w in want.items():
            assert torch.equal(out[n], w), f"replay {k}: {n} differs"


def test_nothing_captured():
    require_gpu()
    from paper_2003_03130_amd import CellBatch, CellmechError
    c = small_sphere_case(1002)
    cb = CellBatch.single(c.x, c.tets)
    with pytest.raises(CellmechError):
        cb.graph_launch()
