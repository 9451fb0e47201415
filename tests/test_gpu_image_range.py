"""epic_image on values near the ends of FP32's range: a grid with one cell set
transforms to that value turned by a phase at every pixel, so nothing may
overflow on the way (1e30; 2.4e38 - 2.4e38 i, whose modulus 3.39e38 still fits a
component) or vanish (1e-30)."""
import numpy as np
import pytest

from helpers import U32
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", [16, 32, 48, 64, 96, 128, 192, 256])
@pytest.mark.parametrize("value", [1e-30, 1e30, 2.4e38 - 2.4e38j])
def test_one_cell(side, value):
    torch = _torch()
    import paper_2609_03027_amd as E
    n_time = 5
    rng = np.random.default_rng(side)
    cells = rng.integers(0, side, size=(n_time, 2))
    cells[0] = (side // 2, side // 2)
    plan = E.Plan(np.zeros((1, 2)), np.array([60e6]), np.array([side], dtype=np.int32), 1)
    grid = torch.zeros((n_time, 1, 1, side, side), dtype=torch.complex64, device="cuda")
    value = complex(np.complex64(value))
    for t, (jy, jx) in enumerate(cells):
        grid[t, 0, 0, jy, jx] = value
    sky = torch.empty_like(grid)
    _say(f"case one cell of {value} on {side}^2")
    E.image(plan, grid, n_time, sky)
    torch.cuda.synchronize()
    got = sky.cpu().numpy()[:, 0, 0]
    k = np.arange(side) - side // 2
    # 2 log2 N levels, each a rotation: the constant within sqrt(2) u and two
    # roundings of at most sqrt(2) u each
    tol = 2 * np.ceil(np.log2(side)) * 3 * np.sqrt(2.0) * U32
    for t, (jy, jx) in enumerate(cells):
        ph = np.add.outer(k * (jy - side // 2), k * (jx - side // 2)) % side
        want = value * np.exp(2j * np.pi * ph / side)
        assert np.isfinite(got[t]).all(), (t, jy, jx)
        err = np.abs(got[t].astype(np.complex128) - want).max() / abs(value)
        assert err <= tol, (t, jy, jx, err, tol)
