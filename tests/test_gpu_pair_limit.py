"""128 x 128 channels whose rows fit 64 with more elements than the paired
kernel's LDS takes (1920): they run one class per item, as integrations, as
frames, with Jones kernels and captured."""
import numpy as np
import pytest

import oracle as O
from helpers import U32, image_errors
from test_gpu_pair import FREQ, _array
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ant,frame_len,jones,graph", [
    (1921, 0, False, False),
    (1921, 0, False, True),
    (1921, 3, False, False),
    (1921, 0, True, False),
    (2500, 0, False, False),
])
def test_more_elements_than_the_pair_takes(n_ant, frame_len, jones, graph):
    torch = _torch()
    import paper_2609_03027_amd as E
    n_time = 6
    rng = np.random.default_rng(n_ant)
    pos = _array("spread", n_ant, rng)
    volt = rng.integers(0, 256, size=(n_time, 1, 2, n_ant), dtype=np.uint8)
    x, j0 = O.grid_geometry(pos, FREQ, 128, k=3)
    w = O.gaussian_kernel(x, j0, 3, 0.5)
    kw = {}
    if jones:
        jm = np.eye(2) + 0.2 * (rng.standard_normal((n_ant, 2, 2)) +
                                1j * rng.standard_normal((n_ant, 2, 2)))
        w = (jm[..., None, None] * w[:, None, None]).astype(np.complex64).astype(np.complex128)
        t = np.stack([w.real, w.imag], axis=-1).astype(np.float32)
        kw = dict(jones=True, kernel_table=t[None])
    _say(f"case {n_ant} elements on 128^2: frames of {frame_len}, jones={jones}, graph={graph}")
    plan = E.Plan(pos, np.array([FREQ]), np.array([128], dtype=np.int32), 2, aperture_n=64, **kw)
    acc = E.Accumulator(plan)
    dv = torch.from_numpy(volt).cuda()
    fl = frame_len or n_time
    out = torch.empty((n_time // fl, plan.info["image_floats"]), dtype=torch.float32, device="cuda")
    if frame_len:
        E.accumulate_frames(plan, acc, dv, fl, out)
    else:
        if graph:
            E.Graph(plan, acc, dv).launch()
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
    e = O.decode_int4(volt[:, 0])
    sky = O.sky(O.grid_jones(e, j0, w, 128) if jones else O.grid(e, j0, w, 128))
    for f in range(n_time // fl):
        got = plan.channel_image(out[f].cpu(), 0).numpy()
        mx, _ = image_errors(got, O.accumulate(sky[f * fl:(f + 1) * fl]))
        assert mx.max() <= tol, (f, mx, tol)
    if not frame_len:
        np.testing.assert_array_equal(autos.cpu().numpy().reshape(-1, 4), O.antenna_autos(e))
