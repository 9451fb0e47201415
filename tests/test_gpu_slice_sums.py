"""The sum over time slices rounds once: 64 slices of one sample each, all of
the same voltages, add up to 64 times the one-sample image bit for bit (a
power of two, so the exact sum needs no rounding; a running FP32 sum rounds at
most odd multiples)."""
import numpy as np
import pytest

from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu

FREQ = 60e6
CELL = 0.5 * 299792458.0 / FREQ


@pytest.mark.parametrize("side,n_pol", [(16, 1), (32, 1), (32, 2), (48, 2), (64, 2), (96, 2)])
def test_slice_sums_round_once(side, n_pol):
    torch = _torch()
    import paper_2609_03027_amd as E
    rng = np.random.default_rng([side, n_pol])
    n_ant, n_time = 20, 64
    pos = rng.uniform(-0.2 * side, 0.2 * side, size=(n_ant, 2)) * CELL
    one = rng.integers(0, 256, size=(1, 1, n_pol, n_ant), dtype=np.uint8)
    _say(f"case equal samples in 64 slices: {side}^2, {n_pol} feeds")
    images = []
    for volt in (one, np.repeat(one, n_time, axis=0)):
        plan = E.Plan(pos, np.array([FREQ]), np.array([side], dtype=np.int32), n_pol, time_slices=64)
        acc = E.Accumulator(plan)
        E.accumulate(plan, acc, volt=torch.from_numpy(volt).cuda())
        img = torch.empty(plan.info["image_floats"], dtype=torch.float32, device="cuda")
        acc.export(img, None)
        torch.cuda.synchronize()
        images.append(img.cpu().numpy())
    np.testing.assert_array_equal(images[1], np.float32(n_time) * images[0])
