"""112 and 90 channels of 128 x 128 leave an eighth and a quarter of the chip idle:
their samples go to two slices of different length (the shorter one's workgroups
take turns on the CUs left), as integrations in two calls and as frames."""
import numpy as np
import pytest

import oracle as O
from helpers import fp32_guard, image_errors
from test_gpu_pair import CELL, FREQ
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_chan,n_time,frame_len", [
    (112, 70, 0), (90, 33, 0), (112, 72, 3), (90, 40, 1),
])
def test_short_last_slice(n_chan, n_time, frame_len):
    torch = _torch()
    import paper_2609_03027_amd as E
    rng = np.random.default_rng([n_chan, n_time])
    n_ant = 9
    pos = rng.uniform(-30.0, 29.0, size=(n_ant, 2)) * CELL
    volt = rng.integers(0, 256, size=(n_time, n_chan, 2, n_ant), dtype=np.uint8)
    _say(f"case {n_chan} channels, {n_time} samples, frames of {frame_len}")
    plan = E.Plan(pos, np.full(n_chan, FREQ), np.full(n_chan, 128, dtype=np.int32), 2, aperture_n=64)
    acc = E.Accumulator(plan)
    dv = torch.from_numpy(volt).cuda()
    floats = plan.info["image_floats"]
    sets = (plan.info["bytes_acc"] - 4 * floats) / (4 * floats)
    assert 2.0 <= sets < 3.0 and 4 * floats * sets <= 97 << 20
    fl = frame_len or n_time
    out = torch.empty((n_time // fl, floats), dtype=torch.float32, device="cuda")
    if frame_len:
        E.accumulate_frames(plan, acc, dv, fl, out)
    else:
        E.accumulate(plan, acc, volt=dv[:-1].contiguous())
        E.accumulate(plan, acc, volt=dv[-1:].contiguous())
        autos = torch.empty(plan.info["autos_ints"], dtype=torch.int32, device="cuda")
        acc.export(out[0], autos)
    torch.cuda.synchronize()
    x, j0 = O.grid_geometry(pos, FREQ, 128, k=3)
    w = O.gaussian_kernel(x, j0, 3, 0.5)
    for c in (0, 8, n_chan - 1):
        e = O.decode_int4(volt[:, c])
        sky = O.sky(O.grid(e, j0, w, 128))
        for f in range(n_time // fl):
            got = plan.channel_image(out[f].cpu(), c).numpy()
            mx, _ = image_errors(got, O.accumulate(sky[f * fl:(f + 1) * fl]))
            assert mx.max() <= fp32_guard(128, 3, fl), (c, f, mx)
        if not frame_len:
            np.testing.assert_array_equal(
                autos.cpu().numpy().reshape(n_chan, n_ant, 4)[c], O.antenna_autos(e))
