"""The packed voltages of the banded path at their edges: element counts around
the four a lane packs, around a workgroup's and past what one sample's buffer
holds, one and two feeds, 4- and 8-bit samples, sample counts around a
workgroup's, several rounds with a remainder, frames, and a channel that is
not banded.  The self terms, which a pass of their own adds here (four elements a
lane where words allow it), are whole numbers and equal the oracle's."""
import numpy as np
import pytest

import oracle as O
from helpers import U32, image_errors
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu

FREQ = 60e6
CELL = 0.5 * 299792458.0 / FREQ
BANDED = -1


@pytest.mark.parametrize("n,n_ant,n_pol,bits,n_time,frame_len,mixed", [
    (64, 1, 2, 4, 1, 0, False),
    (64, 3, 1, 4, 16, 0, False),
    (64, 4, 2, 8, 17, 0, False),
    (64, 255, 2, 8, 15, 0, False),
    (64, 256, 1, 8, 33, 0, False),
    (64, 257, 2, 4, 41, 0, True),
    (64, 250, 2, 4, 15, 5, False),
    (64, 4096, 2, 8, 3, 0, False),
    (64, 4099, 1, 4, 3, 0, False),
    (64, 4100, 2, 4, 3, 0, False),
    (64, 16500, 2, 4, 2, 0, False),
    (64, 16389, 2, 8, 2, 0, False),
    (256, 61, 2, 4, 19, 0, False),
    (512, 130, 2, 4, 18, 0, False),
    (64, 8, 2, 4, 1100, 0, False),      # several time chunks of the self terms
    (64, 5, 1, 8, 1100, 0, False),
])
def test_packed_voltages(n, n_ant, n_pol, bits, n_time, frame_len, mixed, monkeypatch):
    torch = _torch()
    import paper_2609_03027_amd as E
    monkeypatch.setenv("EPIC_BAND_ROUND", "16")   # samples of a round, at most
    rng = np.random.default_rng([n, n_ant, n_pol, bits, n_time])
    # support j0 = floor(x - 1/2) for K = 3, all over the grid
    x = rng.integers(0, n - 2, size=(n_ant, 2)) + 0.5 + rng.uniform(0.0, 0.49, size=(n_ant, 2))
    pos = (x - n / 2.0) * CELL
    n_chan = 2
    if bits == 4:
        volt = rng.integers(0, 256, size=(n_time, n_chan, n_pol, n_ant), dtype=np.uint8)
    else:
        volt = rng.integers(-128, 128, size=(n_time, n_chan, n_pol, n_ant, 2), dtype=np.int8)
    gx, j0 = O.grid_geometry(pos, FREQ, n, k=3)
    w = O.gaussian_kernel(gx, j0, 3, 0.5)
    _say(f"case packed voltages {n}^2: {n_ant} elements x {n_pol} feeds, {bits} bits, "
         f"{n_time} samples, frames of {frame_len}, mixed {mixed}")
    plan = E.Plan(pos, np.full(n_chan, FREQ), np.full(n_chan, n, dtype=np.int32), n_pol,
                  sub_n=[BANDED, 0 if mixed else BANDED], volt_bits=bits)
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
    # taps of a cell, transform, products, time
    tol = (2 * (2 * np.log2(n) + 2 + 4 * cells.max()) + fl) * U32
    for c in range(n_chan):
        e = O.decode_voltages(volt[:, c])
        sky = O.sky(O.grid(e, j0, w, n))
        for f in range(n_time // fl):
            got = plan.channel_image(out[f].cpu(), c).numpy()
            mx, _ = image_errors(got, O.accumulate(sky[f * fl:(f + 1) * fl]))
            assert mx.max() <= tol, (c, f, mx, tol)
    if not frame_len:
        want = np.concatenate([O.antenna_autos(O.decode_voltages(volt[:, c]))
                               for c in range(n_chan)])
        np.testing.assert_array_equal(autos.cpu().numpy().reshape(len(want), -1),
                                      np.asarray(want).reshape(len(want), -1))
