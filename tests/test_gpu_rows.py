"""The row-unfolded kernel (96 x 96 and 48 x 48 grids whose element rows fit half
the side) at its edges: rows that span exactly half the side and one row more
(which takes the general kernel), one sample, slices with a remainder, lists
longer than one batch, element counts around the kernel's threads, frames, and
the largest element count it takes."""
import numpy as np
import pytest

import oracle as O
from helpers import U32, image_errors
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu

FREQ = 60e6
CELL = 0.5 * 299792458.0 / FREQ


@pytest.mark.parametrize("n", [96, 48])
@pytest.mark.parametrize("span,n_ant,n_chan,n_time,frame_len", [
    ("half", 64, 1, 1, 0),
    ("half", 65, 3, 9, 0),
    ("half", 256, 1, 131, 0),
    ("over", 256, 1, 17, 0),
    ("few", 129, 2, 10, 0),
    ("few", 1, 1, 3, 0),
    ("half", 2048, 1, 3, 0),
    ("over", 2049, 1, 2, 0),
    ("half", 100, 2, 12, 4),
    ("over", 100, 1, 10, 5),
])
def test_row_unfolded(n, span, n_ant, n_chan, n_time, frame_len):
    torch = _torch()
    import paper_2609_03027_amd as E
    rng = np.random.default_rng([n, n_ant, n_chan, n_time])
    half = n // 2
    # rows 5 .. 5 + half - 1 (or one more), columns anywhere
    rows = {"half": half, "over": half + 1, "few": 5}[span]
    row0 = rng.integers(5, 5 + rows - 2, size=n_ant)
    row0[0], row0[-1] = 5, 5 + rows - 3
    col0 = rng.integers(0, n - 2, size=n_ant)
    off = rng.uniform(0.0, 0.49, size=(n_ant, 2))
    # support j0 = floor(x - 1/2) for K = 3
    x = np.stack([col0, row0], axis=1) + 0.5 + off
    pos = (x - n / 2.0) * CELL
    volt = rng.integers(0, 256, size=(n_time, n_chan, 2, n_ant), dtype=np.uint8)
    gx, j0 = O.grid_geometry(pos, FREQ, n, k=3)
    assert j0[:, 1].max() - j0[:, 1].min() + 3 == (rows if n_ant > 1 else 3)
    w = O.gaussian_kernel(gx, j0, 3, 0.5)
    _say(f"case row-unfolded {n}^2: {span} span, {n_ant} elements, {n_chan} channels, "
         f"{n_time} samples, frames of {frame_len}")
    plan = E.Plan(pos, np.full(n_chan, FREQ), np.full(n_chan, n, dtype=np.int32), 2)
    acc = E.Accumulator(plan)
    dv = torch.from_numpy(volt).cuda()
    fl = frame_len or n_time
    out = torch.empty((n_time // fl, plan.info["image_floats"]), dtype=torch.float32, device="cuda")
    if frame_len:
        E.accumulate_frames(plan, acc, dv, fl, out)
    else:
        E.accumulate(plan, acc, volt=dv)
        autos = torch.empty(plan.info["autos_ints"], dtype=torch.int32, device="cuda")
        acc.export(out[0], autos)
    torch.cuda.synchronize()
    cells = np.zeros((n, n), dtype=int)
    for jx, jy in j0:
        cells[jy:jy + 3, jx:jx + 3] += 1
    # taps of a cell (and of the cells folded onto it), transform, products, time
    tol = (2 * (14 + 4 * cells.max()) + fl) * U32
    for c in range(n_chan):
        e = O.decode_int4(volt[:, c])
        sky = O.sky(O.grid(e, j0, w, n))
        for f in range(n_time // fl):
            got = plan.channel_image(out[f].cpu(), c).numpy()
            mx, _ = image_errors(got, O.accumulate(sky[f * fl:(f + 1) * fl]))
            assert mx.max() <= tol, (c, f, mx, tol)
    if not frame_len:
        want = np.concatenate([O.antenna_autos(O.decode_int4(volt[:, c])) for c in range(n_chan)])
        np.testing.assert_array_equal(autos.cpu().numpy().reshape(-1, 4), want)
