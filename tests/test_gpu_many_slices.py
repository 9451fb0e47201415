"""A few small grids in up to 64 time slices: fewer samples than slices, as many,
one more (slices of two samples and a short last one) and many, on 16-, 32- and
48-cell grids with one and two feeds."""
import numpy as np
import pytest

import oracle as O
from helpers import U32, image_errors
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu

FREQ = 60e6
CELL = 0.5 * 299792458.0 / FREQ


@pytest.mark.parametrize("n,n_pol,n_chan,n_time", [
    (32, 1, 1, 1), (32, 2, 1, 63), (32, 1, 1, 64), (32, 2, 2, 65), (32, 2, 1, 517),
    (16, 1, 1, 130), (48, 1, 1, 100),
])
def test_many_slices(n, n_pol, n_chan, n_time):
    torch = _torch()
    import paper_2609_03027_amd as E
    n_ant = 23
    rng = np.random.default_rng([n, n_pol, n_chan, n_time])
    x = rng.integers(0, n - 2, size=(n_ant, 2)) + 0.5 + rng.uniform(0.0, 0.49, size=(n_ant, 2))
    pos = (x - n / 2.0) * CELL                              # support j0 = floor(x - 1/2), K = 3
    volt = rng.integers(0, 256, size=(n_time, n_chan, n_pol, n_ant), dtype=np.uint8)
    _say(f"case many slices {n}^2: {n_chan} channels x {n_pol} feeds, {n_time} samples")
    plan = E.Plan(pos, np.full(n_chan, FREQ), np.full(n_chan, n, dtype=np.int32), n_pol)
    acc = E.Accumulator(plan)
    E.accumulate(plan, acc, volt=torch.from_numpy(volt).cuda())
    out = torch.empty(plan.info["image_floats"], dtype=torch.float32, device="cuda")
    autos = torch.empty(plan.info["autos_ints"], dtype=torch.int32, device="cuda")
    acc.export(out, autos)
    torch.cuda.synchronize()
    gx, j0 = O.grid_geometry(pos, FREQ, n, k=3)
    w = O.gaussian_kernel(gx, j0, 3, 0.5)
    cells = np.zeros((n, n), dtype=int)
    for jx, jy in j0:
        cells[jy:jy + 3, jx:jx + 3] += 1
    # taps of a cell (and of those folded onto it), transform, products, time
    tol = (2 * (14 + 4 * cells.max()) + n_time) * U32
    for c in range(n_chan):
        e = O.decode_int4(volt[:, c])
        mx, _ = image_errors(plan.channel_image(out.cpu(), c).numpy(),
                             O.accumulate(O.sky(O.grid(e, j0, w, n))))
        assert mx.max() <= tol, (c, mx, tol)
        want = O.antenna_autos(e)
        np.testing.assert_array_equal(autos.cpu().numpy().reshape(n_chan, n_ant, -1)[c], want)
