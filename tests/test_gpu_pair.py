"""The paired-class kernel (128 x 128 grids whose element rows fit 64) at its
edges: one sample, slices with and without a remainder, rows that span exactly
64, lists of one tap and lists longer than the ones held in registers, element
counts around the 512 and 1024 that a thread's rounds cover, frames cut into
slices, with one kernel per element and with Jones kernels."""
import numpy as np
import pytest

import oracle as O
from helpers import U32, image_errors
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu

FREQ = 60e6
CELL = 0.5 * 299792458.0 / FREQ


def _array(kind, n_ant, rng):
    """Positions whose 3 x 3 supports stay in the central 64 x 64 cells."""
    if kind == "dense":                      # tens of taps per cell
        return rng.uniform(-3.0, 3.0, size=(n_ant, 2)) * CELL
    pos = rng.uniform(-30.4, 29.4, size=(n_ant, 2)) * CELL
    pos[0] = (-31.0 * CELL, -31.0 * CELL)    # first rows 32, last rows 95
    pos[-1] = (30.0 * CELL, 30.0 * CELL)
    return pos


@pytest.mark.parametrize("kind,n_ant,n_chan,n_time,frame_len,jones", [
    ("spread", 1, 1, 1, 0, False),
    ("spread", 64, 1, 1, 0, True),
    ("spread", 256, 1, 33, 0, False),
    ("spread", 256, 3, 130, 0, False),
    ("spread", 511, 2, 9, 0, False),
    ("dense", 513, 1, 17, 0, False),
    ("dense", 1025, 2, 6, 0, False),
    ("spread", 1920, 1, 5, 0, False),
    ("dense", 100, 1, 40, 0, True),
    ("spread", 600, 2, 7, 0, True),
    ("spread", 256, 1, 36, 4, False),
    ("dense", 64, 2, 35, 5, False),
    ("spread", 64, 1, 12, 3, True),
])
def test_paired_classes(kind, n_ant, n_chan, n_time, frame_len, jones):
    torch = _torch()
    import paper_2609_03027_amd as E
    rng = np.random.default_rng([n_ant, n_chan, n_time])
    pos = _array(kind, n_ant, rng)
    freq = np.full(n_chan, FREQ)
    volt = rng.integers(0, 256, size=(n_time, n_chan, 2, n_ant), dtype=np.uint8)
    x, j0 = O.grid_geometry(pos, FREQ, 128, k=3)
    w = O.gaussian_kernel(x, j0, 3, 0.5)
    kw = {}
    if jones:
        jm = np.eye(2) + 0.2 * (rng.standard_normal((n_ant, 2, 2)) +
                                1j * rng.standard_normal((n_ant, 2, 2)))
        w = (jm[..., None, None] * w[:, None, None]).astype(np.complex64).astype(np.complex128)
        t = np.stack([w.real, w.imag], axis=-1).astype(np.float32)
        kw = dict(jones=True, kernel_table=np.broadcast_to(t, (n_chan,) + t.shape))
    _say(f"case paired classes: {kind}, {n_ant} elements, {n_chan} channels, {n_time} samples, "
         f"frames of {frame_len}, jones={jones}")
    plan = E.Plan(pos, freq, np.full(n_chan, 128, dtype=np.int32), 2, aperture_n=64, **kw)
    acc = E.Accumulator(plan)
    dv = torch.from_numpy(volt).cuda()
    floats = plan.info["image_floats"]
    fl = frame_len or n_time
    out = torch.empty((n_time // fl, floats), dtype=torch.float32, device="cuda")
    if frame_len:
        E.accumulate_frames(plan, acc, dv, fl, out)
    else:
        E.accumulate(plan, acc, volt=dv)
        autos = torch.empty(plan.info["autos_ints"], dtype=torch.int32, device="cuda")
        acc.export(out[0], autos)
    torch.cuda.synchronize()
    # a cell's sum of n taps rounds n times (twice with two feeds per grid);
    # transform, products and time sum as in fp32_guard
    cells = np.zeros((128, 128), dtype=int)
    for jx, jy in j0:
        cells[jy:jy + 3, jx:jx + 3] += 1
    tol = (2 * (14 + cells.max() * (2 if jones else 1)) + fl) * U32
    for c in range(n_chan):
        e = O.decode_int4(volt[:, c])
        sky = O.sky(O.grid_jones(e, j0, w, 128) if jones else O.grid(e, j0, w, 128))
        for f in range(n_time // fl):
            got = plan.channel_image(out[f].cpu(), c).numpy()
            mx, _ = image_errors(got, O.accumulate(sky[f * fl:(f + 1) * fl]))
            assert mx.max() <= tol, (c, f, mx, tol)
    if not frame_len:
        want = np.concatenate([O.antenna_autos(O.decode_int4(volt[:, c])) for c in range(n_chan)])
        np.testing.assert_array_equal(autos.cpu().numpy().reshape(-1, 4), want)
