"""Rounds of the FP32 banded path on both sides of the counts from which their
voltages are packed (1000 elements; 2^18 elements x channels x samples), and of those from
which the pack's workgroups are smaller (2048 of them): element
counts that fill words or not, past what one sample's buffer holds, one and two
feeds, 4- and 8-bit samples, a packed round followed by one that is not, frames,
and a captured call."""
import numpy as np
import pytest

import oracle as O
from helpers import U32, image_errors
from test_gpu_band_pack import BANDED, CELL, FREQ
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_ant,n_pol,bits,n_time,round_len,frame_len,graph", [
    (64, 999, 2, 4, 140, 512, 0, False),        # too few elements
    (64, 1000, 2, 4, 131, 512, 0, False),       # 262 000
    (64, 1000, 2, 4, 132, 512, 0, False),       # 264 000: packed
    (64, 1001, 1, 4, 132, 512, 0, False),
    (64, 1027, 2, 8, 130, 512, 0, False),
    (64, 4099, 1, 8, 33, 512, 0, False),
    (64, 1000, 2, 4, 263, 132, 0, False),       # a packed round, then one that is not
    (64, 1000, 2, 4, 264, 132, 12, False),      # frames, two packed rounds
    (64, 1000, 2, 4, 132, 512, 0, True),
    (64, 16384, 2, 8, 8, 512, 0, False),        # 64 KiB a sample and channel
    (64, 16389, 2, 8, 8, 512, 0, False),        # past it: scattered stores
    (64, 32772, 2, 4, 4, 512, 0, False),
    (256, 1100, 2, 4, 120, 512, 0, False),
    (512, 2048, 2, 4, 64, 512, 0, False),
    (64, 1001, 2, 4, 260, 512, 0, False),       # with eight channels: 2080 workgroups
    (64, 1004, 1, 8, 257, 512, 0, False),
])
def test_rounds(n, n_ant, n_pol, bits, n_time, round_len, frame_len, graph, monkeypatch):
    torch = _torch()
    import paper_2609_03027_amd as E
    monkeypatch.setenv("EPIC_BAND_ROUND", str(round_len))
    rng = np.random.default_rng([n, n_ant, n_pol, bits, n_time])
    x = rng.integers(0, n - 2, size=(n_ant, 2)) + 0.5 + rng.uniform(0.0, 0.49, size=(n_ant, 2))
    pos = (x - n / 2.0) * CELL
    n_chan = 8 if n == 64 and n_time in (257, 260) else 2
    if bits == 4:
        volt = rng.integers(0, 256, size=(n_time, n_chan, n_pol, n_ant), dtype=np.uint8)
    else:
        volt = rng.integers(-128, 128, size=(n_time, n_chan, n_pol, n_ant, 2), dtype=np.int8)
    gx, j0 = O.grid_geometry(pos, FREQ, n, k=3)
    w = O.gaussian_kernel(gx, j0, 3, 0.5)
    _say(f"case rounds of {n}^2: {n_ant} elements x {n_pol} feeds, {bits} bits, {n_time} samples "
         f"in rounds of {round_len}, frames of {frame_len}, graph {graph}")
    plan = E.Plan(pos, np.full(n_chan, FREQ), np.full(n_chan, n, dtype=np.int32), n_pol,
                  sub_n=[BANDED] * n_chan, volt_bits=bits)
    acc = E.Accumulator(plan)
    dv = torch.from_numpy(volt).cuda()
    fl = frame_len or n_time
    out = torch.empty((n_time // fl, plan.info["image_floats"]), dtype=torch.float32, device="cuda")
    if frame_len:
        E.accumulate_frames(plan, acc, dv, fl, out)
    elif graph:
        E.Graph(plan, acc, dv).launch()
        acc.export(out[0], None)
    else:
        E.accumulate(plan, acc, volt=dv)
        acc.export(out[0], None)
    torch.cuda.synchronize()
    cells = np.zeros((n, n), dtype=int)
    for jx, jy in j0:
        cells[jy:jy + 3, jx:jx + 3] += 1
    # taps of a cell, transform, products, time
    tol = (2 * (2 * np.log2(n) + 2 + 4 * cells.max()) + fl) * U32
    c = n_chan - 1
    e = O.decode_voltages(volt[:, c])
    got = [plan.channel_image(out[f].cpu(), c).numpy() for f in range(n_time // fl)]
    want = [0.0] * len(got)
    for t0 in range(0, n_time, 4):               # a few skies at a time
        sky = O.sky(O.grid(e[t0:t0 + 4], j0, w, n))
        for f in range(t0 // fl, (t0 + 3) // fl + 1):
            part = sky[max(0, f * fl - t0):max(0, (f + 1) * fl - t0)]
            if f < len(got) and len(part):
                want[f] = want[f] + O.accumulate(part)
    for f, img in enumerate(got):
        mx, _ = image_errors(img, want[f])
        assert mx.max() <= tol, (f, mx, tol)
