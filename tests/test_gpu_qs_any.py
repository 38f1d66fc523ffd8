"""cm_qs_any (is any cell's state column positive) on the GPU: cell counts on
both sides of the workgroup's 256 threads, the one positive entry first, last
and in between, other columns and values that are not positive (zero, negative,
NaN), into pinned and device memory, and its errors."""
import numpy as np
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1000])
def test_any(n):
    require_gpu()
    import torch
    from paper_2003_03130_amd import CellBatch
    from paper_2003_03130_amd import _native as nat
    from paper_2003_03130_amd.cells import _ptr, _stream
    x = np.array([[0.0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]])
    cb = CellBatch.template(n, x, np.array([[0, 1, 2, 3]]))
    pinned = torch.full((1,), 7, dtype=torch.int32, pin_memory=True)
    device = torch.full((1,), 7, dtype=torch.int32, device=cb.device)

    def ask(state, col):
        got = []
        for flag in (pinned, device):
            nat.check(nat.lib().cm_qs_any(cb._h, _ptr(state), col, _ptr(flag), _stream(None)))
            torch.cuda.synchronize()
            got.append(int(flag[0]))
        assert got[0] == got[1]
        return got[0]

    state = torch.zeros(n, 16, dtype=torch.float64, device=cb.device)
    state[:, 3] = 1.0
    state[:, 5], state[:, 6] = -1.0, float("nan")
    assert [ask(state, c) for c in (0, 3, 5, 6, 15)] == [0, 1, 0, 0, 0]
    for c in {0, n // 2, n - 1}:
        state[c, 15] = 1e-300
        assert ask(state, 15) == 1
        state[c, 15] = 0.0
    for bad in (-1, 16):
        assert nat.lib().cm_qs_any(cb._h, _ptr(state), bad, _ptr(pinned), _stream(None)) != 0
    assert nat.lib().cm_qs_any(cb._h, None, 0, _ptr(pinned), _stream(None)) != 0
    assert nat.lib().cm_qs_any(cb._h, _ptr(state), 0, None, _stream(None)) != 0
